// rda_kernels.inl -- gfx950 kernels of the Range Doppler Algorithm and their
// launchers.  Compiled in parts (rda_part_*.hip, SAR_PART = 0..4) so that
// the template instantiations build in parallel: part 0 holds the table
// generators, the non-line kernels and the dispatcher, parts 1-3 the line
// and RCMC kernels for FP32, split-FP16 and split-BF16 butterflies, part 4
// the turn-free strips and the half-storage kernels.  Every kernel is written for
// wave64 CDNA4; lines are kept in registers (16 complex64 per thread) and LDS
// between radix passes.
//
// Kernels (paper: arXiv 2604.03585):
//   k_gen_*          FP64 plan-time tables (twiddles, matched filters with
//                    the IFFT's 1/N folded in, hyperbolic per-bin tables).
//   k_line           FFT -> x H -> IFFT per line, one HBM read and one write
//                    (Sec. II.B; range compression and LFM azimuth
//                    compression, Sec. IV.A steps 1 and 4), or the FFT or IFFT
//                    alone (azimuth FFT of Sec. IV.A step 2; the first/last
//                    dispatch of the unfused comparator, Fig. 1); k_line_pipe
//                    its persistent form for long lines.
//   k_line_tiled,    the range pass into column tiles and the azimuth pass
//   k_line_strip     over strips of them (no corner turn); k_batch_range and
//                    k_batch_strip the same for many scenes.
//   k_line_batch     k_line's lines of many scenes.
//   k_rowmul         the unfused comparator's separate filter multiply.
//   k_corner_turn    LDS-tiled [rows][cols] -> [cols][rows] transpose
//                    (Sec. IV.B).
//   k_rcmc_az,       RCMC (8-tap Kaiser-sinc) + exact-geometry azimuth phase
//   k_rcmc_az2,      + IFFT, fused (Sec. IV.A steps 3-4): one, two and four
//   k_rcmc_rows      output range lines per group of threads.
//   k_rcmc_interp,   the same two steps as separate dispatches for the
//   k_az_phase       unfused comparator.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <initializer_list>
#include <type_traits>

#include "fft_line.hpp"
#include "fft_line_tw.hpp"
#include "mfma_fft.hpp"
#include "rcmc_fit.hpp"
#include "rda_internal.h"

// Every kernel launch of the library.  When sar_time_next_launch has armed
// two events on this thread, the launch records them at the kernel's start
// and end (hipExtLaunchKernel takes the dispatch's own timestamps, so the
// interval is the kernel's duration alone).
#define SAR_LAUNCH(kernel, grid, block, lds, stream, ...)                                  \
    do {                                                                                   \
        hipEvent_t sar_e0_, sar_e1_;                                                       \
        if (sar::take_launch_events(sar_e0_, sar_e1_))                                     \
            hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, sar_e0_, sar_e1_, 0,   \
                                  __VA_ARGS__);                                            \
        else                                                                               \
            hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);             \
    } while (0)

namespace sar {

#if SAR_PART == 0
// ===================================================== FP64 generators
// exp(-2 pi i * num / den) in FP64, num reduced exactly mod den first.
__device__ __forceinline__ float2 twiddle_fp64(long long num, long long den)
{
    long long r = num % den;
    double s, c;
    sincospi(-2.0 * (double)r / (double)den, &s, &c);
    return make_float2((float)c, (float)s);
}

// Per-N Stockham twiddle table (layout in fft_line.hpp, LineGeom::tw_off),
// for radix-E passes followed by one smaller pass.
__global__ void k_gen_twiddles(float2* __restrict__ tw, int n, int e_pts)
{
    int log = 0, rlog = 0;
    while ((1 << log) < n) ++log;
    while ((1 << rlog) < e_pts) ++rlog;
    const int nfull = log / rlog, rem = 1 << (log % rlog);
    const int np = nfull + (rem > 1 ? 1 : 0);
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    int off = 0, ns = 1;
    for (int p = 0; p < np; ++p) {
        const int R = p < nfull ? e_pts : rem;
        if (p >= 1) {
            const int cnt = (R - 1) * ns;
            if (e >= off && e < off + cnt) {
                const int i = (e - off) / ns + 1, jm = (e - off) % ns;
                tw[e] = twiddle_fp64((long long)jm * i, (long long)ns * R);
                return;
            }
            off += cnt;
        }
        ns *= R;
    }
}

// Matched filter H[k] = scale * conj( sum_u exp(j*(sign*pi*K*u^2 - 2*pi*k*u/N)) ),
// u = -L/2 .. L-L/2-1: the DFT of the circularly centred chirp replica,
// evaluated directly (O(N*L)) in FP64 with every phase reduced to turns.
__global__ void k_gen_chirp_filter(float2* __restrict__ H, int n, int len, double K,
                                   int sign, double scale)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    double re = 0.0, im = 0.0;
    const int u0 = -(len / 2), u1 = len - len / 2;
    for (int u = u0; u < u1; ++u) {
        // phase in turns: sign*K*u^2/2 - k*u/n
        double a = (double)sign * 0.5 * K * (double)u * (double)u;
        a -= a >= 0.0 ? floor(a) : -floor(-a);       // exact-ish fraction, |a| < 1
        long long ku = ((long long)k * (long long)u) % n;
        double b = a - (double)ku / (double)n;
        double s, c;
        sincospi(2.0 * b, &s, &c);
        re += c;
        im += s;
    }
    H[k] = make_float2((float)(re * scale), (float)(-im * scale));
}


#endif  // SAR_PART == 0

// ===================================================== line kernels
// FP16 storage of intermediates (the half-storage precision mode): a
// complex sample as two _Float16, with a power-of-two scale per line.
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float2 h2_to_f2(h2_t v, float scale)
{
    return make_float2((float)v.x * scale, (float)v.y * scale);
}
// X: a multiple of the default lines per workgroup (the autotuner's 2x
// candidate of the FP32 line kernels).
template <int N, int X = 1> struct LineLaunch {
    static constexpr int T = LineGeom<N>::T;
    static constexpr int LPW = (T >= 256 ? 1 : 256 / T) * X;   // lines per workgroup
    static constexpr int BLOCK = LPW * T;
    // Register policy of the fused FFT*H*IFFT kernels: the inverse transform
    // may keep the forward passes' twiddles (the same eight values per pass)
    // in registers across the multiply, 16 registers a pass.  Up to 1024
    // points all of them; at 2048, held to 128 VGPRs by line_wpe, pass 1's
    // (with pass 2's as well it spills); from 4096 none: with all but pass
    // 2's the 4096-point kernel (126 VGPRs) took 116 us for 8192 lines, where
    // reading them anew one pass ahead (74 VGPRs) takes 105.
    static constexpr int FRESH_INV = N >= 4096 ? 0xf : (N >= 2048 ? 1 << 2 : 0);
    static constexpr int LDS_BYTES = LPW * LineGeom<N>::LDS * (int)sizeof(float2);
};

// One workgroup per group of LPW lines.
enum LineKind { LK_FUSED = 0, LK_FWD = 1, LK_INV = 2 };

// Minimum waves per SIMD requested for the line kernels: 4 for 1024 points and
// more (FP32 up to 4096, as many workgroups as LDS allows; the split-precision
// ones take 112 to 128 VGPRs; split BF16 below 4096 points 3, for the reads of its
// trailing pass's twiddles), else 2 in the split precisions (130 VGPRs; held to
// 128 they spill; KEEP, see split_may_keep: 135 to 160) and no request in FP32.
template <int N, int PREC, bool KEEP = false> constexpr int line_wpe()
{
    if constexpr (PREC == 0) return N >= 1024 && N <= 4096 ? 4 : 1;
    else return N >= 4096 || (N >= 1024 && PREC == 1 && !KEEP) ? 4 : (N >= 1024 && !KEEP ? 3 : 2);
}

// Split-precision fused lines of 1024 and 2048 points whose workgroups are resident
// in one round at three waves per SIMD (TWP = false there: no table variant exists):
// the inverse transform keeps the forward one's LDS slots and twiddles in registers.
// With a round or less every workgroup's own latency counts (2048 x 1024 LFM scene,
// BF16 37.6 us against 39.4, FP16 37.8 against 39.2; 1024 x 1024 25.8 against 26.8), with
// more of them the fourth wave does (2048 x 2048 64.7 against 62.1).
template <int N, int KIND, int PREC> constexpr bool split_may_keep()
{
    return PREC != PREC_FP32 && KIND == LK_FUSED && (N == 1024 || N == 2048);
}

// Line transform in the requested butterfly precision: FP32 VALU passes, or
// split FP16 / BF16 radix-16 passes on MFMA (twiddles and filters in FP32).
// IN_MF: the input is in the operand layout (split precisions; the output is
// where mf_out).
template <int N, bool INV, int PREC, bool TWP = true, bool SPLIT = false, class F = NoOp,
          bool AHEAD = false, int FRESH = 0, bool IN_MF = false>
__device__ __forceinline__ void fft_any(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                        const float2* __restrict__ tw, int sub, int t,
                                        F&& before_last = F())
{
    if constexpr (PREC == PREC_FP32 && !TWP) {
        if constexpr (FRESH != 0) t = fresh(t);   // the forward passes' would spill
        tw_first::fft_line<N, INV, true, SPLIT>(x, lds, tw, t, before_last);
    } else if constexpr (PREC == PREC_FP32 && AHEAD) {
        fft_line_ahead<N, INV, SPLIT, FRESH>(x, lds, tw, t, before_last);
    } else if constexpr (PREC == PREC_FP32) {
        fft_line<N, INV, SPLIT, FRESH>(x, lds, tw, t, before_last);
    } else {
        using L = LineLaunch<N>;
        fft_line_mfma<N, INV, PREC, L::LPW, L::BLOCK, IN_MF, !TWP && N <= 2048>(x, lds - sub * LineGeom<N>::LDS, tw, sub,
                                                                   t, before_last);
    }
}

// XCD-aware line order: gfx950 hands workgroup b to XCD (b mod 8); giving each
// XCD a contiguous run of line groups keeps neighbouring lines in one L2.
__device__ __forceinline__ int xcd_group(int b, int groups)
{
    if ((groups & 7) != 0) return b;
    return (b & 7) * (groups >> 3) + (b >> 3);
}

// Sample at byte offset `off` from a wave-uniform base.
__device__ __forceinline__ float2 ld_off(const float2* __restrict__ base, uint32_t byte_off)
{
    return *(const float2*)((const char*)base + byte_off);
}

__device__ __forceinline__ float4 buf_ld4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
__device__ __forceinline__ void buf_st(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float2 v)
{
    typedef unsigned int u2_t __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2_t, v), r, voff, soff, 0);
}

// Non-temporal store: for results that no later kernel reads.
__device__ __forceinline__ void buf_st_nt(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float2 v)
{
    typedef unsigned int u2_t __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2_t, v), r, voff, soff, 2);
}
// 16-byte store.  Without a scalar offset: with one the compiler puts no wait
// state between a store of more than 8 bytes and a VALU instruction that writes
// its data registers again, and on gfx950 that store can take the new values (a
// build with such an instruction right behind one store of a turned-back 1024 x
// 2048 image had 16 samples of that store wrong in 5% of the passes).
__device__ __forceinline__ void buf_st4(__amdgpu_buffer_rsrc_t r, uint32_t voff, float4 v)
{
    typedef unsigned int u4_t __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, v), r, voff, 0, 0);
}

// Points t + m*T of a line, or those of the operand layout (MF); `off` is the
// byte offset of the thread's first point from the resource's base.
template <int N, bool MF = false>
__device__ __forceinline__ void load_line(float2 (&x)[line_e(N)], __amdgpu_buffer_rsrc_t src,
                                          uint32_t off)
{
#pragma unroll
    for (int m = 0; m < line_e(N); ++m) x[m] = buf_ld(src, off, mf_step<N, MF>(m) * 8u);
}

template <int N, bool MF = false>
__device__ __forceinline__ void store_line(const float2 (&x)[line_e(N)], __amdgpu_buffer_rsrc_t dst,
                                           uint32_t off)
{
#pragma unroll
    for (int m = 0; m < line_e(N); ++m) buf_st(dst, off, mf_step<N, MF>(m) * 8u, x[m]);
}

// The RCMC pass's stores of its image lines pass by the caches (non-temporal):
// the rows that are still gathered then stay in an XCD's L2, and the image is not
// read again.  Whole hyperbolic scenes over rotating buffers, past the caches
// against through them, us: 1024 x 4096 48.6 v 53.0, 2048 x 4096 93.9 v 99.1, 8192 x
// 2048 236 v 245, 8192 x 8192 952 v 969, 16384 x 1024 263 v 272; split FP16 4096 x
// 4096 244 v 251, half storage 4096 x 8192 370 v 389: better at 40 of 41 sizes from 32
// to 512 MiB.  CACHED: lines of 4096 points in FP32 over more than 64 MiB, where it
// is even or worse (4096 x 2048 97.4 v 101.9, x 4096 198 v 187, x 8192 410 v 410, x
// 16384 812 v 814; 2048 x 8192 192 v 196).  Their azimuth lines come in strips of four
// columns, 32-byte runs, which the last-level cache has to merge, and the next
// scene's strip FFT takes 70 us instead of 52 at 4096 x 4096 when the image went
// past it.
template <int N, bool CACHED = false, bool MF = false>
__device__ __forceinline__ void store_image_line(const float2 (&x)[line_e(N)], __amdgpu_buffer_rsrc_t dst,
                                                 uint32_t off)
{
#pragma unroll
    for (int m = 0; m < line_e(N); ++m) {
        if constexpr (CACHED) buf_st(dst, off, mf_step<N, MF>(m) * 8u, x[m]);
        else buf_st_nt(dst, off, mf_step<N, MF>(m) * 8u, x[m]);
    }
}

// As above, of an image of `bytes` bytes formed by kernels of precision PREC from
// FP32 rows or (HIN) FP16 ones.
template <int N, int PREC, bool HIN, bool MF>
__device__ __forceinline__ void store_image_line(const float2 (&x)[line_e(N)], __amdgpu_buffer_rsrc_t dst,
                                                 uint32_t off, uint32_t bytes)
{
    if (N == 4096 && PREC == PREC_FP32 && !HIN && bytes > (64u << 20))
        store_image_line<N, true, MF>(x, dst, off);
    else
        store_image_line<N, false, MF>(x, dst, off);
}

// Column tiles: the range output between the two passes of the turn-free
// schedules.  Element (m, n) of [na][nr] sits at
//     ((n / 32) na + (m ^ (n / 32 & key_mask))) 32 + n % 32 ,
// i.e. tiles of 32 columns (256-byte rows) one after another.  A strip of
// adjacent azimuth lines then reads its C * 8-byte runs 256 bytes apart instead
// of nr * 8 bytes apart, where (nr a power of two) every row of a strip falls
// into the same few memory channels.  The exclusive or does the same for the
// range pass, whose pieces of one line are na * 256 bytes apart: it moves
// neighbouring tiles' rows to different channels (128 of them, 256 bytes each).
// 4096 x 4096: the strip copy 92 -> 63 us, range + strip FFT 142 -> 114 us,
// the range pass itself unchanged (57 us).
struct TileMap {
    int na;          // rows (azimuth samples)
    int key_mask;    // min(127, na - 1)
};
__host__ __device__ constexpr TileMap tile_map(int na) { return TileMap{na, na < 128 ? na - 1 : 127}; }
constexpr int TILE_COLS = 32;

// Store the points t + m*T of line line0 + sub of the [na][N] array in column
// tiles (LPW lines per workgroup, line0 a multiple of LPW, na one of 64).
template <int N, int LPW>
__device__ __forceinline__ void store_line_tiled(const float2 (&x)[16], float2* out, const TileMap& tm,
                                                 int line0, int sub, int t)
{
    constexpr int T = LineGeom<N>::T, TT32 = T / TILE_COLS;
    const __amdgpu_buffer_rsrc_t ob = buf_rsrc(out, (uint32_t)tm.na * (uint32_t)N * 8u);
    if constexpr (TT32 >= LPW) {
        // tile = t / 32 + m TT32: its low bits meet the lane's part of the row
        // number, the others the workgroup's, so one vector offset serves all m
        const int lo = ((line0 + sub) & (TT32 - 1)) ^ (t / TILE_COLS);
        const uint32_t off = (uint32_t)(((t / TILE_COLS) * tm.na + lo) * TILE_COLS + t % TILE_COLS) * 8u;
        const int hi = line0 & ~(TT32 - 1);
#pragma unroll
        for (int m = 0; m < 16; ++m)
            buf_st(ob, off, (uint32_t)((m * TT32) * tm.na + (hi ^ ((m * TT32) & tm.key_mask))) * (TILE_COLS * 8u),
                   x[m]);
    } else {
        const int line = line0 + sub;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int n = t + m * T, tile = n / TILE_COLS;
            const uint32_t e = (uint32_t)((tile * tm.na + (line ^ (tile & tm.key_mask))) * TILE_COLS + n % TILE_COLS);
            buf_st(ob, e * 8u, 0, x[m]);
        }
    }
}

//  LK_FUSED: out = IFFT(FFT(in) * H)      (H carries the 1/N)
//  LK_FWD:   out = FFT(in) * scale;  LK_INV: out = IFFT_unscaled(in) * scale
// The transform of one line held by its T threads (thread t: points t + m*T;
// split precisions: in the layout of mf_in, left in that of mf_out) with `lds`
// its exchange buffer: FFT * H * IFFT, FFT or IFFT.  TWP: the default transform
// (fft_line), or every twiddle from the table and ahead of the butterflies
// (false), chosen per line length by the autotuner; SPLIT (FP32 forward /
// inverse): the split real/imaginary exchange layout.
template <int N, int KIND, int PREC, bool TWP, bool SPLIT = false>
__device__ __forceinline__ void line_transform(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                               const float2* __restrict__ H,
                                               const float2* __restrict__ tw, float scale,
                                               int sub, int t)
{
    using L = LineLaunch<N>;
    constexpr int E = line_e(N);
    constexpr bool IN = mf_in<N, PREC>(), OUT = mf_out<N, PREC>();
    if constexpr (KIND == LK_FUSED) {
        // the filter is requested just before the last forward pass; lines of
        // 4096 points and more read their twiddles one pass ahead, shorter
        // ones keep the forward passes' for the inverse (see FRESH_INV)
        constexpr bool AHEAD = N >= 4096;
        float2 h[E];
        const __amdgpu_buffer_rsrc_t hb = buf_rsrc(H, N * 8u);
        auto filter = [&] { load_line<N, OUT>(h, hb, (uint32_t)mf_point<N, OUT>(t) * 8u); };
        fft_any<N, false, PREC, TWP, false, decltype(filter)&, AHEAD, 0, IN>(x, lds, tw, sub, t, filter);
#pragma unroll
        for (int m = 0; m < E; ++m) x[m] = c_mul(x[m], h[m]);
        fft_any<N, true, PREC, TWP, false, NoOp, AHEAD, L::FRESH_INV, OUT>(x, lds, tw, sub, t);
    } else {
        fft_any<N, KIND == LK_INV, PREC, TWP, SPLIT, NoOp, true, 0, IN>(x, lds, tw, sub, t);
        if (scale != 1.0f) {
#pragma unroll
            for (int m = 0; m < E; ++m) x[m] = c_scale(x[m], scale);
        }
    }
}

// One group of LPW lines starting at line g * LPW of `in` / `out`.
template <int N, int KIND, int PREC, bool TWP, bool SPLIT = false, int X = 1>
__device__ __forceinline__ void line_group(const float2* in, float2* out, int lines,
                                           const float2* __restrict__ H,
                                           const float2* __restrict__ tw, float scale, int g,
                                           float2* smem)
{
    using L = LineLaunch<N, X>;
    constexpr int E = line_e(N);
    const int sub = threadIdx.x / L::T, t = threadIdx.x % L::T;
    // the group's lines, the last group's only as far as they go: absent
    // lines read zeros and are not stored
    const size_t first = (size_t)g * L::LPW * N;
    const int here = lines - g * L::LPW;
    const uint32_t bytes = (uint32_t)((here < L::LPW ? here : L::LPW) * N) * 8u;
    constexpr bool IN = mf_in<N, PREC>(), OUT = mf_out<N, PREC>();
    float2* lds = smem + sub * LineGeom<N>::LDS;
    float2 x[E];
    load_line<N, IN>(x, buf_rsrc(in + first, bytes), (uint32_t)(sub * N + mf_point<N, IN>(t)) * 8u);
    line_transform<N, KIND, PREC, TWP, SPLIT>(x, lds, H, tw, scale, sub, t);
    store_line<N, OUT>(x, buf_rsrc(out + first, bytes), (uint32_t)(sub * N + mf_point<N, OUT>(t)) * 8u);
}

// The range pass of the turn-free schedules: fused lines stored in column tiles
// (group g of LPW lines of the [na][N] array).
template <int N>
__device__ __forceinline__ void line_tiled_group(const float2* in, float2* out, const float2* __restrict__ H,
                                                 const float2* __restrict__ tw, const TileMap& tm, int g,
                                                 float2* smem)
{
    using L = LineLaunch<N>;
    const int sub = threadIdx.x / L::T, t = threadIdx.x % L::T, line0 = g * L::LPW;
    float2 x[16];
    load_line<N>(x, buf_rsrc(in + (size_t)line0 * N, L::LPW * N * 8u), (uint32_t)(sub * N + t) * 8u);
    line_transform<N, LK_FUSED, PREC_FP32, true>(x, smem + sub * LineGeom<N>::LDS, H, tw, 1.0f, sub, t);
    store_line_tiled<N, L::LPW>(x, out, tm, line0, sub, t);
}

template <int N>
__global__ __launch_bounds__((LineLaunch<N>::BLOCK))
__attribute__((amdgpu_waves_per_eu(line_wpe<N, PREC_FP32>()))) void
k_line_tiled(const float2* in, float2* out, const float2* __restrict__ H,
             const float2* __restrict__ tw, TileMap tm)
{
    extern __shared__ __align__(16) float2 smem[];
    line_tiled_group<N>(in, out, H, tw, tm, blockIdx.x, smem);
}

// ---------------------------------------------------------- column strips
// Turn-free schedules: the azimuth lines of a strip of C adjacent range cells
// are read straight from the range output (column tiles), so no corner turn is
// needed.  Each row of the strip is C consecutive samples; the workgroup reads
// the C x N strip with consecutive lanes on consecutive sample pairs, regroups
// it through LDS into one line per slot of T = N/16 threads, runs the same
// butterflies as k_line (so the results are bit-identical to the turned path)
// and stores each line contiguously: out is [Nr][Na].
//
// What bounds it is how many loads are in flight and what each request brings.
// The line exchange and the regrouping go through half the LDS (fft_line_half)
// at 64 registers per thread, so a CU holds 2048 threads: two workgroups of 4
// lines at 4096 points (one before), which load, transform and store out of
// step.  C: as many lines as 1024 threads take, up to 8 (64-byte runs; 16 lines
// were no faster and left fewer workgroups).  4096 x 4096 strip FFT after a
// range pass: 75 -> 57 us, fused 86 -> 78.
template <int N, int CW = 0> struct StripLaunch {
    static constexpr int T = LineGeom<N>::T;
    static constexpr int C_DEFAULT = (1024 / T) < 8 ? 1024 / T : (T >= 8 ? 8 : 16);
    static constexpr int C = CW ? CW : C_DEFAULT;
    static constexpr int BLOCK = C * T;
    // lines 64 / C floats more than a multiple of 64 apart, which keeps the C samples
    // of a row apart in pairs (32 lanes are served together: two turns)
    static constexpr int STRIDE = (N + N / 16 + 63) / 64 * 64 + 64 / C;
    static constexpr int LDS_BYTES = C * STRIDE * (int)sizeof(float);
    static_assert(N <= 8192 && C >= 2 && C <= 16, "strips of two lines or more");
};

// Source of a strip: rows `row_bytes` apart, row m of it at row m ^ key.
struct StripSrc {
    const float2* base;      // sample (row 0, first column) for key = 0
    uint32_t bytes;          // readable bytes from base
    int key;
};
__device__ __forceinline__ StripSrc strip_source(const float2* in, const TileMap& tm, int cols, int n0)
{
    const int tile = n0 / TILE_COLS;
    StripSrc s;
    s.base = in + (size_t)tile * tm.na * TILE_COLS + n0 % TILE_COLS;
    s.bytes = (uint32_t)((cols / TILE_COLS - tile) * tm.na) * (TILE_COLS * 8u) - (uint32_t)(n0 % TILE_COLS) * 8u;
    s.key = tile & tm.key_mask;
    return s;
}

// Strip g of the scene (uniform per wave), by the C T threads u = 0 .. C T - 1.
// BACK: the lines leave as they came, C samples of every row of out [N][cols]
// (the back-turned image), regrouped through LDS once more.
template <int N, int KIND, int CW, bool BACK>
__device__ __forceinline__ void strip_group(const float2* __restrict__ in, float2* __restrict__ out,
                                            int cols, const TileMap& tm, const float2* __restrict__ H,
                                            const float2* __restrict__ tw, float scale, int g, int u,
                                            float* smem)
{
    using S = StripLaunch<N, CW>;
    constexpr int T = S::T, C = S::C;
    constexpr uint32_t ROW = TILE_COLS * 8u;      // bytes between rows of a tile
    static_assert(KIND == LK_FUSED || KIND == LK_FWD, "fused or forward");
    const int n0 = g * C;
    const StripSrc src = strip_source(in, tm, cols, n0);
    const __amdgpu_buffer_rsrc_t ib = buf_rsrc(src.base, src.bytes);
    // 16-byte loads: lanes take pairs of adjacent columns, C / 2 lanes per row,
    // rows m0 + 2 T p; the row's exclusive or splits into the lane's and the
    // load's part because m0 < 2 T
    static_assert(C % 2 == 0, "pairs of columns");
    const int m0 = u / (C / 2), q = u % (C / 2);
    const uint32_t voff = (uint32_t)(m0 ^ (src.key & (2 * T - 1))) * ROW + (uint32_t)q * 16u;
    float4 v[8];
#pragma unroll
    for (int p = 0; p < 8; ++p)
        v[p] = buf_ld4(ib, voff, (uint32_t)((2 * T * p) ^ (src.key & ~(2 * T - 1))) * ROW);
    const int sub = u / T, t = u % T;
    float* row0 = smem + 2 * q * S::STRIDE;
    float* lds = smem + sub * S::STRIDE;
    float2 x[16];
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        row0[half_in<2 * T, 0>(m0, p)] = v[p].x;
        row0[S::STRIDE + half_in<2 * T, 0>(m0, p)] = v[p].z;
    }
    wg_barrier();
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m].x = lds[half_in<T, 0>(t, m)];
    wg_barrier();
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        row0[half_in<2 * T, 0>(m0, p)] = v[p].y;
        row0[S::STRIDE + half_in<2 * T, 0>(m0, p)] = v[p].w;
    }
    wg_barrier();
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m].y = lds[half_in<T, 0>(t, m)];
    wg_barrier();
    if constexpr (KIND == LK_FUSED) {
        fft_line_half<N, false>(x, lds, tw, t);
        const __amdgpu_buffer_rsrc_t hb = buf_rsrc(H, N * 8u);
#pragma unroll
        for (int m = 0; m < 16; ++m) x[m] = c_mul(x[m], buf_ld(hb, (uint32_t)t * 8u, m * T * 8u));
        fft_line_half<N, true>(x, lds, tw, t);
    } else {
        fft_line_half<N, false>(x, lds, tw, t);
        if (scale != 1.0f) {
#pragma unroll
            for (int m = 0; m < 16; ++m) x[m] = c_scale(x[m], scale);
        }
    }
    if constexpr (!BACK) {
        store_line<N>(x, buf_rsrc(out + (size_t)n0 * N, C * N * 8u), (uint32_t)(sub * N + t) * 8u);
    } else {
#pragma unroll
        for (int m = 0; m < 16; ++m) lds[half_in<T, 0>(t, m)] = x[m].x;
        wg_barrier();
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            v[p].x = row0[half_in<2 * T, 0>(m0, p)];
            v[p].z = row0[S::STRIDE + half_in<2 * T, 0>(m0, p)];
        }
        wg_barrier();
#pragma unroll
        for (int m = 0; m < 16; ++m) lds[half_in<T, 0>(t, m)] = x[m].y;
        wg_barrier();
        const __amdgpu_buffer_rsrc_t ob = buf_rsrc(out + n0, (uint32_t)(N * cols - n0) * 8u);
        const uint32_t off = (uint32_t)(m0 * cols + 2 * q) * 8u;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            v[p].y = row0[half_in<2 * T, 0>(m0, p)];
            v[p].w = row0[S::STRIDE + half_in<2 * T, 0>(m0, p)];
            buf_st4(ob, off + (uint32_t)(2 * T * p * cols) * 8u, v[p]);
        }
    }
}

template <int N, int KIND, int CW = 0, bool BACK = false>
__global__ __launch_bounds__((StripLaunch<N, CW>::BLOCK))
__attribute__((amdgpu_waves_per_eu(N == 512 ? 7 : 8))) void      // 512 points spill at 64 registers
k_line_strip(const float2* __restrict__ in, float2* __restrict__ out, int cols, TileMap tm,
             const float2* __restrict__ H, const float2* __restrict__ tw, float scale)
{
    extern __shared__ __align__(16) float2 smem[];
    strip_group<N, KIND, CW, BACK>(in, out, cols, tm, H, tw, scale,
                                   xcd_group(blockIdx.x, cols / StripLaunch<N, CW>::C), threadIdx.x,
                                   (float*)smem);
}

template <int N, int KIND, int PREC, bool TWP, bool SPLIT = false, int X = 1>
__global__ __launch_bounds__((LineLaunch<N, X>::BLOCK))
__attribute__((amdgpu_waves_per_eu(line_wpe<N, PREC, split_may_keep<N, KIND, PREC>() && !TWP>()))) void
k_line(const float2* in, float2* out, int lines, const float2* __restrict__ H,
       const float2* __restrict__ tw, float scale)
{
    static_assert(!SPLIT || (PREC == PREC_FP32 && KIND != LK_FUSED), "split layout: FP32 FFT only");
    static_assert(X == 1 || PREC == PREC_FP32, "more lines per workgroup: FP32 butterflies only");
    extern __shared__ __align__(16) float2 smem[];
    line_group<N, KIND, PREC, TWP, SPLIT, X>(in, out, lines, H, tw, scale, blockIdx.x, smem);
}

// Persistent form for long lines: a grid of the resident workgroups, each
// walking lines blockIdx.x, + gridDim.x, ...; the next line's loads are issued
// before the inverse transform (fused) or the transform of the current one, so
// they and the previous stores are in flight while it computes.  One 8192- or
// 16384-point line fills half or all of a CU's LDS, so with one line per
// workgroup loads, transform and stores run one after another: 64 Mpx of
// 16384-point fused lines took 315 us where the transform alone needs 176 and
// a copy 190; this form takes 275 (8192 points: 266 -> 237; with the earlier
// transform 393 and 305).  What makes it work:
// nothing in the transforms reads memory (held twiddle reads, see TwAll), so
// no wait of theirs covers the loads of the next line; the loads share one
// address register; every value that enters the loop is pinned, so that the
// loop's first wait does not cover its own stores.
// TILED: stored in column tiles (tm), else line after line.
template <int N, int KIND, bool TILED = false>
__global__ __launch_bounds__(LineGeom<N>::T) __attribute__((amdgpu_waves_per_eu(4))) void
k_line_pipe(const float2* in, float2* out, int lines, const float2* __restrict__ H,
            const float2* __restrict__ tw, float scale, TileMap tm)
{
    constexpr uint32_t BYTES = N * 8u;
    extern __shared__ __align__(16) float2 smem[];
    const int t = threadIdx.x;
    const uint32_t off = (uint32_t)t * 8u;
    TwAll<N> held;
    held.read(tw, t);
    int line = blockIdx.x;
    float2 x[16], nx[16];
    load_line<N>(x, buf_rsrc(in + (size_t)line * N, BYTES), off);
    pin_line(x);
    held.hold();
    for (;;) {
        held.hold();
        const int next = line + (int)gridDim.x;
        const bool more = next < lines;                          // uniform
        const __amdgpu_buffer_rsrc_t nb = buf_rsrc(in + (more ? (size_t)next * N : 0), more ? BYTES : 0u);
        if constexpr (KIND == LK_FUSED) {
            fft_line_held<N, false>(x, smem, held, fresh(t),
                                    [&] { load_line<N>(nx, buf_rsrc(H, BYTES), off); });
#pragma unroll
            for (int m = 0; m < 16; ++m) x[m] = c_mul(x[m], nx[m]);
            __builtin_amdgcn_sched_barrier(0);
            load_line<N>(nx, nb, off);
            __builtin_amdgcn_sched_barrier(0);
            fft_line_held<N, true>(x, smem, held, fresh(t));
        } else {
            load_line<N>(nx, nb, off);
            __builtin_amdgcn_sched_barrier(0);
            fft_line_held<N, KIND == LK_INV>(x, smem, held, fresh(t));
            if (scale != 1.0f) {
#pragma unroll
                for (int m = 0; m < 16; ++m) x[m] = c_scale(x[m], scale);
            }
        }
        if constexpr (TILED) store_line_tiled<N, 1>(x, out, tm, line, 0, t);
        else store_line<N>(x, buf_rsrc(out + (size_t)line * N, BYTES), off);
        if (!more) break;
        line = next;
        __builtin_amdgcn_sched_barrier(0);
        pin_line(nx);
        copy_line(x, nx);
    }
}

// Batched form: the line groups of many scenes (tasks) in one launch.  The
// grid covers min(total groups, resident capacity) workgroups, each walking
// groups gg = blockIdx.x, + gridDim.x, ...; the task of a group is found by
// binary search over the tasks' first-group indices (sorted).
// The task owning line group gg (tasks sorted by group_begin; uniform).
template <class Task>
__device__ __forceinline__ const Task& find_task(const Task* __restrict__ tasks, int ntasks, int gg)
{
    int lo = 0, hi = ntasks - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tasks[mid].group_begin <= gg) lo = mid;
        else hi = mid - 1;
    }
    return tasks[lo];
}

// PERSIST: a grid smaller than the work loops over line groups; otherwise
// one workgroup per line group (no loop, so nothing is hoisted across
// groups and the register footprint equals k_line's).
template <int N, int KIND, int PREC, bool TWP, bool PERSIST>
__global__ __launch_bounds__(LineLaunch<N>::BLOCK)
__attribute__((amdgpu_waves_per_eu(line_wpe<N, PREC>()))) void
k_line_batch(const LineTask* __restrict__ tasks, int ntasks, int total_groups, float scale)
{
    extern __shared__ __align__(16) float2 smem[];
    if constexpr (!PERSIST) {
        const LineTask& tk = find_task(tasks, ntasks, blockIdx.x);
        line_group<N, KIND, PREC, TWP>(tk.in, tk.out, tk.lines, tk.H, tk.tw, scale,
                                       blockIdx.x - tk.group_begin, smem);
    } else {
        for (int gg = blockIdx.x; gg < total_groups; gg += gridDim.x) {
            const LineTask tk = find_task(tasks, ntasks, gg);
            line_group<N, KIND, PREC, TWP>(tk.in, tk.out, tk.lines, tk.H, tk.tw, scale,
                                           gg - tk.group_begin, smem);
            __syncthreads();                      // LDS reuse by the next group
        }
    }
}

#if SAR_PART == 4
// Batched turn-free scenes: the two passes of every scene, whatever its line
// length, are two launches.  The groups of a pass are independent and as large
// as each other (4096 points of range lines, 8192 of strips), so a switch on the
// task's length serves all of them with the same threads and LDS.
// What bounds them: memory, once the launch is long enough.  Before, each line
// length had its own launch per pass and a corner turn lay between, all too short
// to fill the chip or to hide their start and end: 24 scenes of 128 to 1024 points
// a side (78 MB moved per pass) took 54.7 us in nine launches, 33.8 in these two.
// (64-point strips are left out: eight of them side by side take 66 KiB of LDS,
// two workgroups per CU for every scene of the launch.)
#define SAR_BATCH_LENGTHS(X) X(128) X(256) X(512) X(1024) X(2048) X(4096)

constexpr int BATCH_RANGE_BLOCK = 256;
#define SAR_LDS(N) LineLaunch<N>::LDS_BYTES,
constexpr int batch_max(std::initializer_list<int> l)
{
    int m = 0;
    for (int v : l) m = v > m ? v : m;
    return m;
}
constexpr int BATCH_RANGE_LDS = batch_max({SAR_BATCH_LENGTHS(SAR_LDS)});
#undef SAR_LDS

__global__ __launch_bounds__(BATCH_RANGE_BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void
k_batch_range(const SceneTask* __restrict__ tasks, int ntasks)
{
    extern __shared__ __align__(16) float2 smem[];
    const SceneTask& tk = find_task(tasks, ntasks, blockIdx.x);
    const int g = blockIdx.x - tk.group_begin;
    const TileMap tm = tile_map(tk.other);
    switch (tk.n) {
#define SAR_CASE(N)                                                              \
    case N:                                                                      \
        static_assert(LineLaunch<N>::BLOCK == BATCH_RANGE_BLOCK, "one block size"); \
        line_tiled_group<N>(tk.in, tk.out, tk.H, tk.tw, tm, g, smem);            \
        break;
        SAR_BATCH_LENGTHS(SAR_CASE)
#undef SAR_CASE
    }
}

// 512 threads: strips as wide as they take up to the default width, several side
// by side for short lines (whole waves each, so a strip's base is wave-uniform).
constexpr int BATCH_STRIP_BLOCK = 512;
template <int N> struct BatchStrip {
    static constexpr int T = LineGeom<N>::T, D = StripLaunch<N>::C_DEFAULT;
    static constexpr int C = BATCH_STRIP_BLOCK / T < D ? BATCH_STRIP_BLOCK / T : D;
    static constexpr int PER_WG = BATCH_STRIP_BLOCK / (C * T);
    static constexpr int LDS_BYTES = PER_WG * StripLaunch<N, C>::LDS_BYTES;
    static_assert(C * T % 64 == 0, "whole waves per strip");
    static_assert(BATCH_STRIP_MIN % (C * PER_WG) == 0, "no strip beyond the last column");
};
#define SAR_LDS(N) BatchStrip<N>::LDS_BYTES,
constexpr int BATCH_STRIP_LDS = batch_max({SAR_BATCH_LENGTHS(SAR_LDS)});
#undef SAR_LDS

template <int N>
__device__ __forceinline__ void batch_strip_group(const SceneTask& tk, int g, float* smem)
{
    using B = BatchStrip<N>;
    using S = StripLaunch<N, B::C>;
    const int k = __builtin_amdgcn_readfirstlane(threadIdx.x / S::BLOCK);
    strip_group<N, LK_FUSED, B::C, false>(tk.in, tk.out, tk.other, tile_map(N), tk.H, tk.tw, 1.0f,
                                          g * B::PER_WG + k, threadIdx.x % S::BLOCK,
                                          smem + k * (S::LDS_BYTES / 4));
}

__global__ __launch_bounds__(BATCH_STRIP_BLOCK) __attribute__((amdgpu_waves_per_eu(6))) void
k_batch_strip(const SceneTask* __restrict__ tasks, int ntasks, int total)
{
    extern __shared__ __align__(16) float2 smem[];
    const int gg = xcd_group(blockIdx.x, total);
    const SceneTask& tk = find_task(tasks, ntasks, gg);
    const int g = gg - tk.group_begin;
    switch (tk.n) {
#define SAR_CASE(N)                                \
    case N:                                        \
        batch_strip_group<N>(tk, g, (float*)smem); \
        break;
        SAR_BATCH_LENGTHS(SAR_CASE)
#undef SAR_CASE
    }
}
#endif  // SAR_PART == 4

#if SAR_PART == 0
// out[r][k] = in[r][k] * H[k]  (unfused comparator's multiply dispatch)
__global__ __launch_bounds__(256) void k_rowmul(const float4* in, float4* out, long long n_pairs,
                                                int n, const float2* __restrict__ H)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < n_pairs; p += stride) {
        float4 a = in[p];
        const int k = (int)((2 * p) & (n - 1));
        const float2 h0 = H[k], h1 = H[k + 1];
        const float2 r0 = c_mul(make_float2(a.x, a.y), h0);
        const float2 r1 = c_mul(make_float2(a.z, a.w), h1);
        out[p] = make_float4(r0.x, r0.y, r1.x, r1.y);
    }
}

// ===================================================== corner turn
constexpr int TT = 64;

// Batched corner turn: the 64 x 64 tiles of many matrices in one launch.
// Whole 64 x 64 tiles only (rows and cols multiples of 64): every global
// access moves 16 bytes (two complex samples).
// LDS map: element (r, c) of the tile sits at column c ^ ((r >> 1) & 31) of
// row r (no pad).  A bank holds 4 bytes and 64 banks span 32 samples, so a
// sample's banks depend on its column mod 32.  The read phase has lane tx
// take rows 2tx and 2tx+1 at one column c: the swizzle gives the 32 lanes
// 32 different columns mod 32 (with a pad the even rows share 16), and the
// 32 KiB tile lets five workgroups share a CU's LDS instead of four.
__device__ __forceinline__ int turn_swz(int r, int c) { return c ^ ((r >> 1) & 31); }

// Tiles gt = blockIdx.x, + gridDim.x, ... (the launcher keeps gridDim.x <=
// tiles): the next tile's loads are issued before the current tile leaves
// LDS, so they overlap its stores; its LDS writes wait for those loads only
// (vector-memory operations complete in issue order, the stores came after).
// `more` is uniform per workgroup.
__device__ __forceinline__ void turn_tile_to_lds(float2 (*tile)[TT], const float4 (&v)[TT / 8], int tx,
                                                 int ty)
{
#pragma unroll
    for (int i = 0; i < TT / 8; ++i) {
        const int r = ty + 8 * i;
        tile[r][turn_swz(r, 2 * tx)] = make_float2(v[i].x, v[i].y);
        tile[r][turn_swz(r, 2 * tx + 1)] = make_float2(v[i].z, v[i].w);
    }
}

__global__ __launch_bounds__(256) void k_corner_turn_x2(const float4* __restrict__ in,
                                                        float4* __restrict__ out, int rows,
                                                        int cols, int tiles)
{
    __shared__ float2 tile[TT][TT];
    const int tiles_c = cols / TT;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int cols2 = cols / 2, rows2 = rows / 2;
    int gt = blockIdx.x;
    float4 v[TT / 8];
    {
        const int r0 = (gt / tiles_c) * TT, c0 = (gt % tiles_c) * TT;
#pragma unroll
        for (int i = 0; i < TT / 8; ++i) v[i] = in[(size_t)(r0 + ty + 8 * i) * cols2 + c0 / 2 + tx];
    }
    turn_tile_to_lds(tile, v, tx, ty);
    wg_barrier();
    for (;;) {
        const int r0 = (gt / tiles_c) * TT, c0 = (gt % tiles_c) * TT;
        const int next = gt + (int)gridDim.x;
        const bool more = next < tiles;
        if (more) {
            const int nr0 = (next / tiles_c) * TT, nc0 = (next % tiles_c) * TT;
#pragma unroll
            for (int i = 0; i < TT / 8; ++i)
                v[i] = in[(size_t)(nr0 + ty + 8 * i) * cols2 + nc0 / 2 + tx];
        }
#pragma unroll
        for (int i = 0; i < TT / 8; ++i) {
            const int c = ty + 8 * i;
            const float2 a = tile[2 * tx][turn_swz(2 * tx, c)], b = tile[2 * tx + 1][turn_swz(2 * tx + 1, c)];
            out[(size_t)(c0 + c) * rows2 + r0 / 2 + tx] = make_float4(a.x, a.y, b.x, b.y);
        }
        if (!more) break;
        wg_barrier();                             // every read done before the next writes
        turn_tile_to_lds(tile, v, tx, ty);
        wg_barrier();
        gt = next;
    }
}

// Any rows and cols (odd ones start rows on 8-byte boundaries): TR x 64 tiles,
// one workgroup of 4 TR threads each, two samples per access (16 bytes at 8-byte alignment,
// which global memory instructions take) and turn_swz's conflict-free LDS
// map; only tiles on the ragged edges test every sample.
// What bounds it: HBM (3000 x 5001, 240 MB moved: 49 us at the rate of a large
// copy).  One sample per access in a padded tile took 63.7 us there, this form
// 51.1; persistent workgroups that load ahead took 54.4 to 56.2 (eight
// accesses per thread and five workgroups per CU already cover the latency).
// TR = 128 writes runs of 1 KiB: where the output's rows do not start on
// 64-byte boundaries each run ends inside a line at both sides, and half as
// many runs leave half as many torn lines.
typedef float turn_f4 __attribute__((ext_vector_type(4), aligned(8)));
template <int TR>
__global__ __launch_bounds__(4 * TR) void k_corner_turn(const float2* __restrict__ in,
                                                        float2* __restrict__ out, int rows, int cols)
{
    __shared__ float2 tile[TR][TT];
    constexpr int OP = TR / 2;                    // threads per output run
    const int tiles_c = (cols + TT - 1) / TT;
    const int r0 = (int)(blockIdx.x / tiles_c) * TR, c0 = (int)(blockIdx.x % tiles_c) * TT;
    const bool inside = r0 + TR <= rows && c0 + TT <= cols;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    turn_f4 v[8];
    if (inside) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            v[i] = *(const turn_f4*)(in + (size_t)(r0 + ty + TR / 8 * i) * cols + c0 + 2 * tx);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = r0 + ty + TR / 8 * i, c = c0 + 2 * tx;
            const float2* p = in + (size_t)r * cols + c;
            float2 a = make_float2(0.f, 0.f), b = a;
            if (r < rows && c < cols) a = p[0];
            if (r < rows && c + 1 < cols) b = p[1];
            v[i] = turn_f4{a.x, a.y, b.x, b.y};
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = ty + TR / 8 * i;
        tile[r][turn_swz(r, 2 * tx)] = make_float2(v[i].x, v[i].y);
        tile[r][turn_swz(r, 2 * tx + 1)] = make_float2(v[i].z, v[i].w);
    }
    __syncthreads();
    const int ox = threadIdx.x & (OP - 1), oy = threadIdx.x / OP;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = oy + 8 * i;
        const float2 a = tile[2 * ox][turn_swz(2 * ox, c)], b = tile[2 * ox + 1][turn_swz(2 * ox + 1, c)];
        float2* p = out + (size_t)(c0 + c) * rows + r0 + 2 * ox;
        if (inside)
            *(turn_f4*)p = turn_f4{a.x, a.y, b.x, b.y};
        else if (c0 + c < cols) {
            if (r0 + 2 * ox < rows) p[0] = a;
            if (r0 + 2 * ox + 1 < rows) p[1] = b;
        }
    }
}

// k_corner_turn_x2 for 4-byte elements (FP16 pairs): whole 64 x 64 tiles,
// every global access moves two elements (8 bytes).
__global__ __launch_bounds__(256) void k_corner_turn_b4(const uint2* __restrict__ in,
                                                        uint2* __restrict__ out, int rows, int cols)
{
    __shared__ uint32_t tile[TT][TT + 1];
    const int tiles_c = cols / TT;
    const int tr = blockIdx.x / tiles_c, tc = blockIdx.x % tiles_c;
    const int r0 = tr * TT, c0 = tc * TT;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int cols2 = cols / 2, rows2 = rows / 2;
#pragma unroll
    for (int i = 0; i < TT / 8; ++i) {
        const int r = ty + 8 * i;
        const uint2 v = in[(size_t)(r0 + r) * cols2 + c0 / 2 + tx];
        tile[r][2 * tx] = v.x;
        tile[r][2 * tx + 1] = v.y;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TT / 8; ++i) {
        const int c = ty + 8 * i;
        out[(size_t)(c0 + c) * rows2 + r0 / 2 + tx] = make_uint2(tile[2 * tx][c], tile[2 * tx + 1][c]);
    }
}

__global__ __launch_bounds__(256) void k_corner_turn_batch(const TurnTask* __restrict__ tasks,
                                                           int ntasks, int total_tiles)
{
    // every task is whole 64 x 64 tiles (plan sizes are powers of two >= 64);
    // the tile's LDS map is k_corner_turn_x2's
    __shared__ float2 tile[TT][TT];
    for (int gt = blockIdx.x; gt < total_tiles; gt += gridDim.x) {
        int lo = 0, hi = ntasks - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tasks[mid].tile_begin <= gt) lo = mid;
            else hi = mid - 1;
        }
        const TurnTask tk = tasks[lo];
        const int b = gt - tk.tile_begin;
        const int tiles_c = tk.cols / TT;
        const int r0 = (b / tiles_c) * TT, c0 = (b % tiles_c) * TT;
        const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
        const float4* in = (const float4*)tk.in;
        float4* out = (float4*)tk.out;
        const int cols2 = tk.cols / 2, rows2 = tk.rows / 2;
#pragma unroll
        for (int i = 0; i < TT / 8; ++i) {
            const int r = ty + 8 * i;
            const float4 v = in[(size_t)(r0 + r) * cols2 + c0 / 2 + tx];
            tile[r][turn_swz(r, 2 * tx)] = make_float2(v.x, v.y);
            tile[r][turn_swz(r, 2 * tx + 1)] = make_float2(v.z, v.w);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TT / 8; ++i) {
            const int c = ty + 8 * i;
            const float2 a = tile[2 * tx][turn_swz(2 * tx, c)];
            const float2 bb = tile[2 * tx + 1][turn_swz(2 * tx + 1, c)];
            out[(size_t)(c0 + c) * rows2 + r0 / 2 + tx] = make_float4(a.x, a.y, bb.x, bb.y);
        }
        __syncthreads();
    }
}

#endif  // SAR_PART == 0

// ===================================================== RCMC
// (weights and their tables: rcmc_fit.hpp)
// The kernels copy the 12 KiB table of quadratics into LDS with the intervals 7
// vectors (28 floats) apart: the lanes of a wave read random intervals, and with an
// odd stride in 16-byte units the same vector of different intervals falls into
// every bank group, where a stride of 6 reaches only half of them (twice the bank
// conflicts).  The seventh vector of each interval is padding and never read.
constexpr int RCMC_LDS_STRIDE = 28;
constexpr int RCMC_LDS_FLOATS = RCMC_INTERVALS * RCMC_LDS_STRIDE;

#if SAR_PART == 0
// One thread per interval: block 0 the quadratics, block 1 the cubics.
__global__ void k_gen_rcmc_table(float* __restrict__ tab, double beta)
{
    const int b = threadIdx.x;
    if (blockIdx.x == 0 && b < RCMC_INTERVALS)
        rcmc_fit<2>(tab + b * RCMC_PER_INTERVAL, b, RCMC_INTERVALS, 0.0, beta);
    if (blockIdx.x == 1 && b < RROWS_INTERVALS)
        rcmc_fit<3>(tab + RCMC_TAB + b * RROWS_PER_INTERVAL, b, RROWS_INTERVALS, RROWS_MARGIN, beta);
}

#endif  // SAR_PART == 0

struct RcmcArgs {
    const double* stretch;   // 1/D_k - 1 per Doppler bin
    const double* rate;      // 2 D_k / lambda per Doppler bin
    const float* table;      // RCMC_TAB + RROWS_TAB weight coefficients (global)
    double r_near;
    double stretch_max;      // max_k stretch_k (|f| = 1/2)
    double x_per_bin;        // lambda / (2 v Na): x_k = signed bin * x_per_bin
    double two_over_lam;     // 2 / lambda
    int nr;
    const int* row_exp;      // half storage: per-row exponents of the FP16 input
};

// The per-bin geometry from the bin index: f_k in fftfreq order,
// x = lambda f / (2 v), D = sqrt(1 - x^2), stretch = 1/D - 1, rate = 2 D / lambda.
// r = 1/D comes from the hardware reciprocal square root r0 (about 2^-24) refined
// in FP64 by r = r0 (1 + e/2 + 3 e^2 / 8), e = 1 - D^2 r0^2, whose error is of
// third order (full double precision), so stretch = r - 1 has an absolute error
// near 1e-16; the RCMC shift R0 * stretch needs it to 1e-12.  The plan's tables
// use the same function.
__device__ __forceinline__ void bin_geometry_x(double x, double two_over_lam, double& stretch,
                                               double& rate)
{
    const double a = fma(-x, x, 1.0);               // D^2
    const double r0 = __builtin_amdgcn_rsq(a);
    const double e = fma(-a * r0, r0, 1.0);
    const double r = fma(r0 * e, fma(e, 0.375, 0.5), r0);
    stretch = r - 1.0;
    rate = (a * r) * two_over_lam;                  // D = a / sqrt(a)
}

__device__ __forceinline__ void bin_geometry(const RcmcArgs& ra, int k, int na, double& stretch,
                                             double& rate)
{
    const int kk = k < na / 2 ? k : k - na;
    bin_geometry_x((double)kk * ra.x_per_bin, ra.two_over_lam, stretch, rate);
}

#if SAR_PART == 0
// Hyperbolic per-Doppler-bin tables (the unfused and one-row kernels read
// them; the two-row kernel computes the same values in place):
// stretch = 1/D - 1, rate = 2 D / lambda (azimuth phase in turns per cell).
__global__ void k_gen_hyper_tables(double* __restrict__ stretch, double* __restrict__ rate,
                                   int na, double x_per_bin, double two_over_lam)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= na) return;
    const int kk = k < na / 2 ? k : k - na;
    bin_geometry_x((double)kk * x_per_bin, two_over_lam, stretch[k], rate[k]);
}
#endif

// Global table (PER floats per interval) -> LDS (STRIDE floats per interval);
// lds_tab holds INTERVALS * STRIDE floats.
template <int STRIDE = RCMC_LDS_STRIDE, int PER = RCMC_PER_INTERVAL, int INTERVALS = RCMC_INTERVALS>
__device__ __forceinline__ void load_rcmc_table(float* __restrict__ lds_tab,
                                                const float* __restrict__ tab, int tid, int nthreads,
                                                float scale = 1.0f)
{
    static_assert(PER % 4 == 0 && STRIDE % 4 == 0, "16-byte copies");
    constexpr int V = PER / 4, VS = STRIDE / 4;
    for (int i = tid; i < INTERVALS * V; i += nthreads) {
        const float4 v = ((const float4*)tab)[i];
        ((float4*)lds_tab)[(i / V) * VS + i % V] =
            make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
    }
}

// sum_t w_t(x) a_t with the weights from the LDS table.
__device__ __forceinline__ float2 rcmc_combine(float x, const float* __restrict__ tab,
                                               const float2 (&a)[8])
{
    const float xf = x * (float)RCMC_INTERVALS;
    const int b = min((int)xf, RCMC_INTERVALS - 1);
    const float u = xf - (float)b;
    const float4* p = (const float4*)(tab + __mul24(b, RCMC_LDS_STRIDE));
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int h = 0; h < 2; ++h) {                 // taps 4h .. 4h+3: three vectors
        float c[12];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const float4 v = p[3 * h + i];
            c[4 * i] = v.x;
            c[4 * i + 1] = v.y;
            c[4 * i + 2] = v.z;
            c[4 * i + 3] = v.w;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int t = 4 * h + q;
            const float w = fmaf(fmaf(c[3 * q + 2], u, c[3 * q + 1]), u, c[3 * q]);
            acc.x = fmaf(w, a[t].x, acc.x);
            acc.y = fmaf(w, a[t].y, acc.y);
        }
    }
    return acc;
}

// RCMC output y[n][k] from range-Doppler A[Nr][Na]:
//   R0 = r_near + n, s = R0 * stretch_k, i0 = n + floor(s), x = frac(s),
//   y = sum_t w_t(x) A[i0 + t][k] over t = -3..4 (rows outside [0, Nr) add 0).
// `interior` promises that every tap row is inside the scene (checked by
// the caller per line), which removes the per-tap bounds tests.
__device__ __forceinline__ void rcmc_shift(double R0, int n, double stretch, float& x, int& i0)
{
    const double s = R0 * stretch;
    const double fl = floor(s);
    x = (float)(s - fl);
    // shifts beyond +-2^30 cells read nothing but stay defined integers
    i0 = n + (int)fmax(-1073741824.0, fmin(fl, 1073741824.0));
}

__device__ __forceinline__ float2 rcmc_gather(const float2* __restrict__ A, int na, int nr, int k,
                                              float x, int i0, const float* __restrict__ tab,
                                              bool interior)
{
    float2 a[8];
    if (interior) {
        const uint32_t step = (uint32_t)na * 8u;
        uint32_t off = ((uint32_t)(i0 - 3) * (uint32_t)na + (uint32_t)k) * 8u;
#pragma unroll
        for (int i = 0; i < 8; ++i, off += step) a[i] = ld_off(A, off);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = i0 + i - 3;
            a[i] = (r >= 0 && r < nr) ? A[(size_t)r * na + k] : make_float2(0.f, 0.f);
        }
    }
    return rcmc_combine(x, tab, a);
}

template <int TAPS>
__device__ __forceinline__ float2 rcmc_value(const float2* __restrict__ A, int na, int n, int k,
                                             const RcmcArgs& ra, const float* __restrict__ tab,
                                             bool interior)
{
    if constexpr (TAPS == 0) {
        return ld_off(A, ((uint32_t)n * (uint32_t)na + (uint32_t)k) * 8u);
    } else {
        float x;
        int i0;
        rcmc_shift(ra.r_near + (double)n, n, ra.stretch[k], x, i0);
        return rcmc_gather(A, na, ra.nr, k, x, i0, tab, interior);
    }
}

// exp(+j 2 pi ph) * scale: the phase in turns is reduced to [-1/2, 1/2] in FP64,
// then the hardware sine/cosine (argument in turns, max abs error 1.3e-7 there,
// measured on gfx950) evaluate it.
__device__ __forceinline__ float2 turns_to_phasor(double ph)
{
    const float f = (float)(ph - rint(ph));
    return make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
}
__device__ __forceinline__ float2 turns_to_phasor(double ph, float scale)
{
    return c_scale(turns_to_phasor(ph), scale);
}

__device__ __forceinline__ float2 az_phase_of(double R0, double rate, float scale)
{
    return turns_to_phasor(R0 * rate, scale);
}

__device__ __forceinline__ float2 az_phase(const RcmcArgs& ra, int n, int k, float scale)
{
    return az_phase_of(ra.r_near + (double)n, ra.rate[k], scale);
}

// Every tap row of output line n lies inside [0, Nr).
__device__ __forceinline__ bool rcmc_interior(const RcmcArgs& ra, int n)
{
    const double smax = (ra.r_near + (double)n) * ra.stretch_max;
    return n >= 3 && (double)n + smax + 6.0 <= (double)(ra.nr - 1);
}

// Samples y[m] = RCMC(n, k_m) * phase_m for the 16 columns k_m = t + m*T
// of one thread, all tap rows inside the scene.  The eight gathers of
// column m+1 are in flight while column m is combined (vector-memory loads
// complete in order, so the wait for column m leaves m+1's loads pending).
// The eight tap samples A[i0 - 3 + i][k].  EDGE: rows outside [0, nr) are
// read at a clamped (valid) row and replaced by zero, without branches.
template <int N, bool EDGE>
__device__ __forceinline__ void rcmc_gather8(float2 (&a)[8], const float2* __restrict__ A, int k,
                                             int i0, int nr)
{
    if constexpr (!EDGE) {
        constexpr uint32_t step = (uint32_t)N * 8u;
        uint32_t off = ((uint32_t)(i0 - 3) * (uint32_t)N + (uint32_t)k) * 8u;
#pragma unroll
        for (int i = 0; i < 8; ++i, off += step) a[i] = ld_off(A, off);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = i0 - 3 + i;
            const int rc = min(max(r, 0), nr - 1);
            const float2 v = ld_off(A, ((uint32_t)rc * (uint32_t)N + (uint32_t)k) * 8u);
            const bool in = (r >= 0) & (r < nr);
            a[i] = make_float2(in ? v.x : 0.f, in ? v.y : 0.f);
        }
    }
}

// Samples y[m] = RCMC(n, k_m) * phase_m for the 16 columns k_m = t + m*T
// of one thread.  The gathers of column m+1 are in flight while column m is
// combined (vector-memory loads complete in order, so waiting for column m
// leaves m+1's loads pending); sched_barrier(0) keeps the scheduler from
// hoisting every gather to the top, which would need ~256 registers.
template <int N, bool EDGE>
__device__ __forceinline__ void rcmc_row(float2 (&x)[line_e(N)], const float2* __restrict__ A, int t,
                                         int nr, const float (&xs)[line_e(N)], const int (&i0s)[line_e(N)],
                                         const float2 (&ph)[line_e(N)], const float* __restrict__ tab)
{
    constexpr int T = LineGeom<N>::T;
    constexpr int E = line_e(N);
    float2 a0[8], a1[8];
    rcmc_gather8<N, EDGE>(a0, A, t, i0s[0], nr);
#pragma unroll
    for (int m = 0; m < E; m += 2) {
        rcmc_gather8<N, EDGE>(a1, A, t + (m + 1) * T, i0s[m + 1], nr);
        __builtin_amdgcn_sched_barrier(0);
        x[m] = c_mul(rcmc_combine(xs[m], tab, a0), ph[m]);
        __builtin_amdgcn_sched_barrier(0);
        if (m + 2 < E) rcmc_gather8<N, EDGE>(a0, A, t + (m + 2) * T, i0s[m + 2], nr);
        __builtin_amdgcn_sched_barrier(0);
        x[m + 1] = c_mul(rcmc_combine(xs[m + 1], tab, a1), ph[m + 1]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int N, int TAPS, int PREC>
__global__ __launch_bounds__(LineLaunch<N>::BLOCK) void
k_rcmc_az(const float2* __restrict__ A, float2* __restrict__ out, RcmcArgs ra,
               const float2* __restrict__ tw)
{
    using L = LineLaunch<N>;
    constexpr int E = line_e(N);
    extern __shared__ __align__(16) float2 smem[];
    // The weight table and the line buffers share LDS: the table is only read
    // while the RCMC samples are formed, before the first FFT exchange.
    float* tab = (float*)smem;
    static_assert(L::LDS_BYTES >= RCMC_LDS_FLOATS * (int)sizeof(float), "table fits the line LDS");
    const int lines = ra.nr;
    const int groups = (lines + L::LPW - 1) / L::LPW;
    const int g = xcd_group(blockIdx.x, groups);
    const int sub = threadIdx.x / L::T, t = threadIdx.x % L::T;
    const int n = g * L::LPW + sub;
    const bool live = n < lines;
    float2* lds = smem + sub * LineGeom<N>::LDS;
    constexpr float scale = 1.0f / (float)N;
    const double R0 = ra.r_near + (double)n;

    // per-Doppler-bin quantities first: their loads overlap the table copy
    float xs[E];
    int i0s[E];
    float2 ph[E];
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int k = t + m * L::T;
        ph[m] = az_phase_of(R0, ra.rate[k], scale);
        if constexpr (TAPS != 0) rcmc_shift(R0, n, ra.stretch[k], xs[m], i0s[m]);
    }
    if constexpr (TAPS != 0) {
        load_rcmc_table(tab, ra.table, threadIdx.x, L::BLOCK);
        __syncthreads();
    }
    float2 x[E];
    if (!live) {
#pragma unroll
        for (int m = 0; m < E; ++m) x[m] = make_float2(0.f, 0.f);
    } else if constexpr (TAPS == 0) {
#pragma unroll
        for (int m = 0; m < E; ++m)
            x[m] = c_mul(ld_off(A, ((uint32_t)n * (uint32_t)N + (uint32_t)(t + m * L::T)) * 8u), ph[m]);
    } else if (rcmc_interior(ra, n)) {
        rcmc_row<N, false>(x, A, t, ra.nr, xs, i0s, ph, tab);
    } else {
        rcmc_row<N, true>(x, A, t, ra.nr, xs, i0s, ph, tab);
    }
    if constexpr (TAPS != 0) __syncthreads();     // table reads done before LDS reuse
    fft_any<N, true, PREC>(x, lds, tw, sub, t);
    const uint32_t bytes = (uint32_t)(min(L::LPW, lines - g * L::LPW) * N) * 8u;   // absent lines dropped
    constexpr bool OUT = mf_out<N, PREC>();
    store_line<N, OUT>(x, buf_rsrc(out + (size_t)g * L::LPW * N, bytes),
                       (uint32_t)(sub * N + mf_point<N, OUT>(t)) * 8u);
}

// Two output rows n, n+1 per line slot.  For each column their 8-tap
// windows start at i0(n) - 3 and i0(n+1) - 3 with i0(n+1) - i0(n) = 1 + d,
// d in {0, 1} (requires stretch < 1), so ten rows i0(n) - 3 .. i0(n) + 6
// cover both: 10 gathers for 2 samples instead of 16.  The per-bin
// geometry is computed, not loaded, so the gathers of the next column can be
// issued before the current column is combined without a load-to-load chain.
// Range-Doppler rows stored as FP16 pairs, row r scaled by 2^-ex[r].
struct HalfRows {
    const h2_t* a;
    const int* ex;
};

template <int N, bool EDGE>
__device__ __forceinline__ void rcmc_gather10(float2 (&w)[10], const HalfRows& A, int k, int i0,
                                              int nr)
{
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        const int r = i0 - 3 + i;
        const int rc = EDGE ? min(max(r, 0), nr - 1) : r;
        const h2_t v = *(const h2_t*)((const char*)A.a + ((uint32_t)rc * (uint32_t)N + (uint32_t)k) * 4u);
        const float2 f = h2_to_f2(v, ldexpf(1.0f, A.ex[rc]));
        const bool in = !EDGE || ((r >= 0) & (r < nr));
        w[i] = make_float2(in ? f.x : 0.f, in ? f.y : 0.f);
    }
}

template <int N, bool EDGE>
__device__ __forceinline__ void rcmc_gather10(float2 (&w)[10], const float2* __restrict__ A,
                                              int k, int i0, int nr)
{
    if constexpr (!EDGE) {
        constexpr uint32_t step = (uint32_t)N * 8u;
        uint32_t off = ((uint32_t)(i0 - 3) * (uint32_t)N + (uint32_t)k) * 8u;
#pragma unroll
        for (int i = 0; i < 10; ++i, off += step) w[i] = ld_off(A, off);
    } else {
#pragma unroll
        for (int i = 0; i < 10; ++i) {
            const int r = i0 - 3 + i;
            const int rc = min(max(r, 0), nr - 1);
            const float2 v = ld_off(A, ((uint32_t)rc * (uint32_t)N + (uint32_t)k) * 8u);
            const bool in = (r >= 0) & (r < nr);
            w[i] = make_float2(in ? v.x : 0.f, in ? v.y : 0.f);
        }
    }
}

struct ColPair {
    float xa, xb;        // fractional positions for rows n, n+1
    int i0;              // i0(n)
    bool d;              // i0(n+1) - i0(n) == 2
    float2 pa, pb;       // azimuth phases (with 1/Na) for rows n, n+1
};

// Row n+1 continues row n: its shift is s + stretch and its phase (turns)
// ph + rate, both in FP64 (the same values as R0 * stretch and R0 * rate
// with R0 = r_near + n + 1, up to one rounding).
__device__ __forceinline__ ColPair col_pair(const RcmcArgs& ra, int n, int k, int na, float scale)
{
    double stretch, rate;
    bin_geometry(ra, k, na, stretch, rate);
    const double R0 = ra.r_near + (double)n;
    ColPair c;
    const double sa = R0 * stretch, sb = sa + stretch;
    const double fa = floor(sa), fb = floor(sb);
    c.xa = (float)(sa - fa);
    c.xb = (float)(sb - fb);
    // shifts beyond +-2^30 cells read nothing but stay defined integers
    c.i0 = n + (int)fmax(-1073741824.0, fmin(fa, 1073741824.0));
    c.d = (fb - fa) != 0.0;                       // i0(n+1) - i0(n) == 2
    const double pa = R0 * rate;
    c.pa = turns_to_phasor(pa, scale);
    c.pb = turns_to_phasor(pa + rate, scale);
    return c;
}

template <int N, bool EDGE>
__device__ __forceinline__ void rcmc_pair_combine(float2& ya, float2& yb, const ColPair& c,
                                                  const float2 (&w)[10],
                                                  const float* __restrict__ tab)
{
    float2 ta[8], tb[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        ta[i] = w[i];
        tb[i] = c.d ? w[i + 2] : w[i + 1];
    }
    ya = c_mul(rcmc_combine(c.xa, tab, ta), c.pa);
    yb = c_mul(rcmc_combine(c.xb, tab, tb), c.pb);
}

// Columns t + m * S (m < C) of rows n, n+1 of A (FP32 rows, or HalfRows); MF: the
// columns of the operand layout, t the thread's first.
template <int N, bool EDGE, int C = line_e(N), int S = LineGeom<N>::T, class Src = const float2*, bool MF = false>
__device__ __forceinline__ void rcmc_rows2(float2 (&xa)[C], float2 (&xb)[C], Src A,
                                           const RcmcArgs& ra, int n, int t,
                                           const float* __restrict__ tab)
{
    constexpr int E = C;
    auto col = [&](int m) { return t + (MF ? mf_step<N, MF>(m) : m * S); };
    static_assert(E % 2 == 0, "columns are processed in pairs");
    constexpr float scale = 1.0f / (float)N;
    // two named buffers, alternated by column parity (no register copies)
    ColPair c0 = col_pair(ra, n, t, N, scale), c1;
    float2 w0[10], w1[10];
    rcmc_gather10<N, EDGE>(w0, A, t, c0.i0, ra.nr);
#pragma unroll
    for (int m = 0; m < E; m += 2) {
        c1 = col_pair(ra, n, col(m + 1), N, scale);
        rcmc_gather10<N, EDGE>(w1, A, col(m + 1), c1.i0, ra.nr);
        __builtin_amdgcn_sched_barrier(0);
        rcmc_pair_combine<N, EDGE>(xa[m], xb[m], c0, w0, tab);
        __builtin_amdgcn_sched_barrier(0);
        if (m + 2 < E) {
            c0 = col_pair(ra, n, col(m + 2), N, scale);
            rcmc_gather10<N, EDGE>(w0, A, col(m + 2), c0.i0, ra.nr);
        }
        __builtin_amdgcn_sched_barrier(0);
        rcmc_pair_combine<N, EDGE>(xa[m + 1], xb[m + 1], c1, w1, tab);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// HIN: A holds FP16 rows with per-row exponents ra.row_exp (half storage).
template <int N, int PREC, bool HIN = false>
__global__ __launch_bounds__(LineLaunch<N>::BLOCK) void
k_rcmc_az2(const void* __restrict__ A_, float2* __restrict__ out, RcmcArgs ra,
           const float2* __restrict__ tw)
{
    using SrcT = typename std::conditional<HIN, HalfRows, const float2*>::type;
    SrcT A;
    if constexpr (HIN) A = HalfRows{(const h2_t*)A_, ra.row_exp};
    else A = (const float2*)A_;
    using L = LineLaunch<N>;
    constexpr bool IN = mf_in<N, PREC>(), OUT = mf_out<N, PREC>();
    constexpr int E = line_e(N);
    extern __shared__ __align__(16) float2 smem[];
    float* tab = (float*)smem;                    // shares LDS with the line buffers
    static_assert(L::LDS_BYTES >= RCMC_LDS_FLOATS * (int)sizeof(float), "table fits the line LDS");
    const int pairs = ra.nr / 2;
    const int groups = (pairs + L::LPW - 1) / L::LPW;
    const int g = xcd_group(blockIdx.x, groups);
    const int sub = threadIdx.x / L::T, t = threadIdx.x % L::T;
    const int pr = g * L::LPW + sub;
    const bool live = pr < pairs;
    const int n = 2 * pr;
    float2* lds = smem + sub * LineGeom<N>::LDS;
    load_rcmc_table(tab, ra.table, threadIdx.x, L::BLOCK);
    __syncthreads();
    float2 xa[E], xb[E];
    if (!live) {
#pragma unroll
        for (int m = 0; m < E; ++m) xa[m] = xb[m] = make_float2(0.f, 0.f);
    } else {
        const double smax = (ra.r_near + (double)n + 1.0) * ra.stretch_max;
        if (n >= 3 && (double)n + 1.0 + smax + 6.0 <= (double)(ra.nr - 1))
            rcmc_rows2<N, false, line_e(N), LineGeom<N>::T, SrcT, IN>(xa, xb, A, ra, n, mf_point<N, IN>(t), tab);
        else
            rcmc_rows2<N, true, line_e(N), LineGeom<N>::T, SrcT, IN>(xa, xb, A, ra, n, mf_point<N, IN>(t), tab);
    }
    __syncthreads();                              // table reads done before LDS reuse
    fft_any<N, true, PREC, true, false, NoOp, true, 0, IN>(xa, lds, tw, sub, t);
    // the group's pairs of rows (absent ones are not stored)
    const uint32_t bytes = (uint32_t)(min(L::LPW, pairs - g * L::LPW) * 2 * N) * 8u;
    const __amdgpu_buffer_rsrc_t ob = buf_rsrc(out + (size_t)(2 * g * L::LPW) * N, bytes);
    const uint32_t off = (uint32_t)(2 * sub * N + mf_point<N, OUT>(t)) * 8u;
    const uint32_t image = (uint32_t)ra.nr * N * 8u;
    store_image_line<N, PREC, HIN, OUT>(xa, ob, off, image);
    fft_any<N, true, PREC, true, false, NoOp, true, 0, IN>(xb, lds, tw, sub, t);
    store_image_line<N, PREC, HIN, OUT>(xb, ob, off + N * 8u, image);
}

// Four output rows n .. n + 3 per group of threads, for geometries whose shift
// changes little from row to row (stretch up to RCMC_ROWS_STRETCH_MAX).  Up to 2048
// points the group has 4T threads (T = N/16): a thread interpolates four columns of
// the four rows, the rows meet in LDS and their IFFTs run side by side.  At 4096 and 8192 points it has 2T threads and
// works in two rounds: the first two rows' samples go to LDS as they are formed,
// the others wait in registers.  The FP64 geometry, the gathers and the table
// reads are shared by four samples:
//   * twelve rows i0 - 3 .. i0 + 8 cover the four windows;
//   * the shifts s + j stretch, j < 4, lie close together, so one interval (that
//     of their middle) of a table fitted for it serves all rows (RROWS_MARGIN);
//   * where a shift crosses a cell boundary between the rows (a wave vote; one
//     wave in ten) the rows take their own windows and intervals.
// Rows beyond the scene read as zero by the buffer's bounds; only the first
// rows of the scene have rows before it, and take the EDGE form, where every
// row's offset is formed by itself (a negative one is beyond the bounds too).
//
// Bound by VALU issue, at 8192 points by L2 (the rows in flight of an XCD no
// longer fit it).  Against two rows per thread with two buffers of gathers
// (k_rcmc_az2: 157 registers, three waves per SIMD; twice the FP64 work and four
// times the table reads per sample), alone, from HBM: 4096^2 101 -> 74 us, 8192
// x 4096 212 -> 162, 2048 x 1024 20.6 -> 11.8, 1024 x 4096 25 -> 17, 256 x 4096
// 23 -> 7.8.  (At 4096 points one workgroup of 1024 threads per CU took 79.)
template <int N> struct RcmcRows {
    static constexpr int T = LineGeom<N>::T;
    static_assert(N <= 8192, "two lines and the table fit LDS");
    static constexpr int SIDE = N <= 2048 ? 4 : 2;               // rows whose IFFTs run side by side
    static constexpr int ROUNDS = 4 / SIDE;
    static constexpr int R = 4;                                  // rows per group
    static constexpr int S = SIDE * T;                           // threads per group
    static constexpr int C = N / S;                              // columns per thread
    static constexpr int G = S >= 256 ? 1 : 256 / S;             // groups per workgroup
    static constexpr int BLOCK = S * G;
    static constexpr int LINES = SIDE * G * LineGeom<N>::LDS * (int)sizeof(float2);
    // intervals an odd number of 16-byte units apart, see RCMC_LDS_STRIDE
    static constexpr int STRIDE = RROWS_PER_INTERVAL + 4;
    static constexpr int TABLE = RROWS_INTERVALS * STRIDE * (int)sizeof(float);
    // one round: the table shares LDS with the lines, which are written after
    // its last read; two: the first round's rows go to LDS as they are formed
    static constexpr int LDS_BYTES = ROUNDS == 2 ? LINES + TABLE : (LINES > TABLE ? LINES : TABLE);
    static_assert(LDS_BYTES <= 160 * 1024 && (ROUNDS == 1 || G == 1), "one workgroup per CU at least");
};

// HIN: FP16 rows, row r scaled by 2^-exponent[r].
template <bool HIN> struct RcmcSrc {
    __amdgpu_buffer_rsrc_t rows, exponents;
};

template <int N, int ROWS, bool EDGE, bool HIN>
__device__ __forceinline__ void rcmc_gather_rows(float2 (&w)[ROWS], const RcmcSrc<HIN>& A, int first, int k)
{
    constexpr uint32_t B = HIN ? 4u : 8u, ROW = N * B;
    const uint32_t off = (uint32_t)(first * N + k) * B;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const uint32_t vo = EDGE ? off + i * ROW : off, so = EDGE ? 0 : i * ROW;
        if constexpr (HIN) {
            const h2_t v = __builtin_bit_cast(h2_t, __builtin_amdgcn_raw_buffer_load_b32(A.rows, vo, so, 0));
            const int e = (int)__builtin_amdgcn_raw_buffer_load_b32(
                A.exponents, EDGE ? (uint32_t)(first + i) * 4u : (uint32_t)first * 4u, EDGE ? 0 : i * 4u, 0);
            w[i] = h2_to_f2(v, ldexpf(1.0f, e));
        } else {
            w[i] = buf_ld(A.rows, vo, so);
        }
    }
}

__device__ __forceinline__ float rrows_weight(float4 cf, float v)
{
    return fmaf(fmaf(fmaf(cf.w, v, cf.z), v, cf.y), v, cf.x);
}

// sum_t w_t(x) a_t, x on its own interval.
template <int STRIDE>
__device__ __forceinline__ float2 rrows_combine(float x, const float* tab, const float2 (&a)[8])
{
    const float xf = x * (float)RROWS_INTERVALS;
    const int b = min((int)xf, RROWS_INTERVALS - 1);
    const float v = xf - (float)b;
    const float4* q = (const float4*)(tab + __mul24(b, STRIDE));
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float wt = rrows_weight(q[t], v);
        acc.x = fmaf(wt, a[t].x, acc.x);
        acc.y = fmaf(wt, a[t].y, acc.y);
    }
    return acc;
}

// The samples of columns u + m * S: the last SIDE rows' in y, the first round's
// (of two) in the line buffers `lines`.
template <int N, bool EDGE, bool HIN>
__device__ __forceinline__ void rcmc_rows_columns(float2 (&y)[RcmcRows<N>::SIDE][RcmcRows<N>::C],
                                                  const RcmcSrc<HIN>& A, const RcmcArgs& ra, int n, int u,
                                                  const float* tab, float2* lines)
{
    using L = RcmcRows<N>;
    constexpr int R = L::R, ROWS = R + 8;
    const double R0 = ra.r_near + (double)n;
#pragma unroll
    for (int m = 0; m < L::C; ++m) {
        const int k = fresh(u) + m * L::S;
        double stretch, rate;
        bin_geometry(ra, k, N, stretch, rate);
        const double s = R0 * stretch, f = floor(s), ph = R0 * rate;
        float x[R];                               // fractions against row n's cell
#pragma unroll
        for (int j = 0; j < R; ++j) x[j] = (float)(fma((double)j, stretch, s) - f);
        // cells past the scene's end read nothing wherever they are
        const int i0 = n + (int)fmin(f, 32768.0);
        float2 w[ROWS];
        rcmc_gather_rows<N, ROWS, EDGE, HIN>(w, A, i0 - 3, k);
        __builtin_amdgcn_sched_barrier(0);
        if (m == 0) __syncthreads();              // the table is in LDS
        float2 acc[R];
        if (__builtin_amdgcn_ballot_w64(x[R - 1] >= 1.0f) == 0) {
            // one interval for all rows
            const int b = min((int)(0.5f * (x[0] + x[R - 1]) * (float)RROWS_INTERVALS), RROWS_INTERVALS - 1);
            const float fb = (float)b;
            float v[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                v[j] = fmaf(x[j], (float)RROWS_INTERVALS, -fb);
                acc[j] = make_float2(0.f, 0.f);
            }
            const float4* q = (const float4*)(tab + __mul24(b, L::STRIDE));
#pragma unroll
            for (int h = 0; h < 2; ++h) {         // taps 4h .. 4h+3
                float4 cf[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) cf[i] = q[4 * h + i];
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float wt = rrows_weight(cf[i], v[j]);
                        const float2 a = w[4 * h + i + j];
                        acc[j].x = fmaf(wt, a.x, acc[j].x);
                        acc[j].y = fmaf(wt, a.y, acc[j].y);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const bool d = j > 0 && x[j] >= 1.0f;            // the window starts one row later
                float2 a[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) a[i] = d ? w[i + j + 1 < ROWS ? i + j + 1 : 0] : w[i + j];
                acc[j] = rrows_combine<L::STRIDE>(d ? x[j] - 1.0f : x[j], tab, a);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float2 v = c_mul(acc[j], turns_to_phasor(fma((double)j, rate, ph)));
            if (j < R - L::SIDE) lines[j * LineGeom<N>::LDS + lds_in<L::S, 0>(u, m)] = v;
            else y[j - (R - L::SIDE)][m] = v;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// HIN: A holds FP16 rows with per-row exponents ra.row_exp (half storage).
// PREC: butterflies of the IFFT.
template <int N, bool HIN = false, int PREC = PREC_FP32>
__global__ __launch_bounds__(RcmcRows<N>::BLOCK)
__attribute__((amdgpu_waves_per_eu(4))) void
k_rcmc_rows(const void* __restrict__ A, float2* __restrict__ out, RcmcArgs ra,
            const float2* __restrict__ tw)
{
    using L = RcmcRows<N>;
    constexpr int T = L::T, S = L::S, R = L::R, SIDE = L::SIDE, LL = LineGeom<N>::LDS;
    extern __shared__ __align__(16) float2 smem[];
    float* tab = (float*)smem;
    float2* lines = smem + (L::ROUNDS == 2 ? L::TABLE / (int)sizeof(float2) : 0);
    const int g = xcd_group(blockIdx.x, ra.nr / (R * L::G));
    const int gi = threadIdx.x / S, u = threadIdx.x % S;
    const int n0 = g * L::G * R, n = n0 + gi * R;                // n0 uniform
    const uint32_t bytes = (uint32_t)ra.nr * N * 8u;
    RcmcSrc<HIN> ab;
    ab.rows = buf_rsrc(A, HIN ? bytes / 2 : bytes);
    if constexpr (HIN) ab.exponents = buf_rsrc(ra.row_exp, (uint32_t)ra.nr * 4u);
    // the weights carry the IFFT's 1/N (a power of two: exact)
    load_rcmc_table<L::STRIDE, RROWS_PER_INTERVAL, RROWS_INTERVALS>(tab, ra.table + RCMC_TAB, threadIdx.x,
                                                                    L::BLOCK, 1.0f / (float)N);
    float2 y[SIDE][L::C];
    if (n0 >= 4) rcmc_rows_columns<N, false, HIN>(y, ab, ra, n, u, tab, lines);
    else rcmc_rows_columns<N, true, HIN>(y, ab, ra, n, u, tab, lines);
    const __amdgpu_buffer_rsrc_t ob = buf_rsrc(out, bytes);
    const int line = threadIdx.x / T, t = threadIdx.x % T;       // row n0 + line (of a round)
    float2* lds = lines + line * LL;
#pragma unroll
    for (int r = 0; r < L::ROUNDS; ++r) {
        wg_barrier();                             // table reads, or the first round's writes, done
        if (r == L::ROUNDS - 1) {
#pragma unroll
            for (int j = 0; j < SIDE; ++j)
#pragma unroll
                for (int m = 0; m < L::C; ++m) lines[(gi * SIDE + j) * LL + lds_in<S, 0>(u, m)] = y[j][m];
            wg_barrier();
        }
        constexpr bool IN = mf_in<N, PREC>(), OUT = mf_out<N, PREC>();
        float2 x[16];
        const int p0 = mf_point<N, IN>(t);
#pragma unroll
        for (int m = 0; m < 16; ++m)
            x[m] = lds[IN ? lds_slot<0>(p0 + mf_step<N, IN>(m)) : lds_in<T, 0>(t, m)];
        wg_barrier();
        if constexpr (PREC == PREC_FP32)
            fft_line<N, true>(x, lds, tw, fresh(t));
        else
            fft_line_mfma<N, true, PREC, L::BLOCK / T, L::BLOCK, IN>(x, lines, tw, line, t);
        const uint32_t off = (uint32_t)((n0 + r * SIDE + line) * N + mf_point<N, OUT>(t)) * 8u;
        store_image_line<N, PREC, HIN, OUT>(x, ob, off, bytes);
    }
}

// The same two rows per workgroup on 2T threads (FP32, T = N/16 <= 512):
// the interpolation is spread over all 2T threads (E/2 columns each, half
// the accumulator registers of k_rcmc_az2), the two rows then meet in LDS
// and their IFFTs run side by side, one per half of the workgroup.  LDS:
// two line buffers (the weight table shares the first).
template <int N>
__global__ __launch_bounds__(2 * LineGeom<N>::T) void
k_rcmc_az2w(const float2* __restrict__ A, float2* __restrict__ out, RcmcArgs ra,
            const float2* __restrict__ tw)
{
    using G = LineGeom<N>;
    constexpr int T = G::T, E = line_e(N), C = E / 2, S = 2 * T;
    static_assert(S <= 1024, "two line slots per workgroup");
    extern __shared__ __align__(16) float2 smem[];
    float* tab = (float*)smem;
    static_assert(2 * G::LDS * (int)sizeof(float2) >= RCMC_LDS_FLOATS * (int)sizeof(float),
                  "table fits the two line buffers");
    const int pairs = ra.nr / 2;
    const int pr = xcd_group(blockIdx.x, pairs);
    const int n = 2 * pr;
    const int u = threadIdx.x;
    load_rcmc_table(tab, ra.table, u, S);
    __syncthreads();
    float2 ya[C], yb[C];
    const double smax = (ra.r_near + (double)n + 1.0) * ra.stretch_max;
    if (n >= 3 && (double)n + 1.0 + smax + 6.0 <= (double)(ra.nr - 1))
        rcmc_rows2<N, false, C, S>(ya, yb, A, ra, n, u, tab);
    else
        rcmc_rows2<N, true, C, S>(ya, yb, A, ra, n, u, tab);
    __syncthreads();                              // table reads done before LDS reuse
    float2* row_a = smem;
    float2* row_b = smem + G::LDS;
#pragma unroll
    for (int m = 0; m < C; ++m) {
        row_a[lds_in<S, 0>(u, m)] = ya[m];
        row_b[lds_in<S, 0>(u, m)] = yb[m];
    }
    __syncthreads();
    const int sub = u / T, t = u % T;
    float2* lds = smem + sub * G::LDS;
    float2 x[E];
#pragma unroll
    for (int m = 0; m < E; ++m) x[m] = lds[lds_in<T, 0>(t, m)];
    __syncthreads();                              // reads done before the IFFT writes
    fft_line<N, true>(x, lds, tw, t);
    store_line<N>(x, buf_rsrc(out + (size_t)n * N, 2 * N * 8u), (uint32_t)(sub * N + t) * 8u);
}

#if SAR_PART == 0
// Unfused comparator: RCMC interpolation alone (grid-stride, one sample per
// thread per iteration).
template <int TAPS>
__global__ __launch_bounds__(256) void k_rcmc_interp(const float2* __restrict__ A,
                                                     float2* __restrict__ out, int na, RcmcArgs ra)
{
    __shared__ __align__(16) float tab[RCMC_LDS_FLOATS];
    if constexpr (TAPS != 0) {
        load_rcmc_table(tab, ra.table, threadIdx.x, 256);
        __syncthreads();
    }
    const long long total = (long long)ra.nr * na;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const int n = (int)(e / na), k = (int)(e % na);
        out[e] = rcmc_value<TAPS>(A, na, n, k, ra, tab, false);
    }
}

// Unfused comparator: azimuth phase multiply exp(+j 2 pi frac(R0 rate_k)) * scale.
__global__ __launch_bounds__(256) void k_az_phase(const float2* __restrict__ in,
                                                  float2* __restrict__ out, int na, RcmcArgs ra,
                                                  float scale)
{
    const long long total = (long long)ra.nr * na;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const int n = (int)(e / na), k = (int)(e % na);
        out[e] = c_mul(in[e], az_phase(ra, n, k, scale));
    }
}

#endif  // SAR_PART == 0

#if SAR_PART == 4
// ===================================================== half storage (FP32 math)
// Largest |re|, |im| of one line's samples (the line's T threads: aligned
// lane segments of a wave when T < 64, else whole waves combined through
// `scratch`, 16 floats of LDS that no thread still reads).
template <int N>
__device__ __forceinline__ float line_absmax(const float2 (&x)[line_e(N)], float* scratch, int sub)
{
    using L = LineLaunch<N>;
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < line_e(N); ++i) m = fmaxf(m, fmaxf(fabsf(x[i].x), fabsf(x[i].y)));
    constexpr int W = L::T < 64 ? L::T : 64;
#pragma unroll
    for (int off = 1; off < W; off <<= 1) m = fmaxf(m, __shfl_xor(m, off));
    if constexpr (L::T > 64) {
        constexpr int WPL = L::T / 64;            // waves per line
        static_assert(L::BLOCK / 64 <= 16, "scratch holds one float per wave");
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        __syncthreads();
        if (lane == 0) scratch[wave] = m;
        __syncthreads();
        m = 0.f;
#pragma unroll
        for (int w = 0; w < WPL; ++w) m = fmaxf(m, scratch[sub * WPL + w]);
    }
    return m;
}

// Exponent e of a line whose largest component is amax: the stored values
// x * 2^-e have their largest component in [2^14, 2^15) (FP16 holds up to
// 65504); empty, non-finite or all-zero lines keep e = 0.
__device__ __forceinline__ int half_exponent(float amax)
{
    if (!(amax > 0.f) || !(amax < INFINITY)) return 0;
    return max(ilogbf(amax) - 14, -100);
}

// FP32 line transform with FP16 storage on either side.
//  IN_H:  `in` holds lines of FP16 pairs; point j of every line carries the
//         scale 2^ex_in[j] (the exponent of the range line the point came
//         from, after the corner turn);
//  OUT_H: `out` receives FP16 pairs x * 2^-e, e = ex_out[line] chosen per
//         line by half_exponent; else `out` is complex64.
template <int N, int KIND, bool IN_H, bool OUT_H>
__global__ __launch_bounds__(LineLaunch<N>::BLOCK)
__attribute__((amdgpu_waves_per_eu(line_wpe<N, PREC_FP32>()))) void
k_line_hs(const void* __restrict__ in, void* __restrict__ out, int lines,
          const float2* __restrict__ H, const float2* __restrict__ tw,
          const int* __restrict__ ex_in, int* __restrict__ ex_out)
{
    using L = LineLaunch<N>;
    constexpr int E = line_e(N);
    extern __shared__ __align__(16) float2 smem[];
    const int groups = (lines + L::LPW - 1) / L::LPW;
    const int g = xcd_group(blockIdx.x, groups);
    const int sub = threadIdx.x / L::T, t = threadIdx.x % L::T;
    const int line = g * L::LPW + sub;
    const bool live = line < lines;
    const size_t first = (size_t)g * L::LPW * N;                 // uniform
    const uint32_t off = (uint32_t)(sub * N + t);                // samples from `first`
    float2* lds = smem + sub * LineGeom<N>::LDS;
    float2 x[E];
    if (live) {
        if constexpr (IN_H) {
            const h2_t* src = (const h2_t*)in + first;
#pragma unroll
            for (int m = 0; m < E; ++m)
                x[m] = h2_to_f2(*(const h2_t*)((const char*)(src + m * L::T) + off * 4u),
                                ldexpf(1.0f, *(const int*)((const char*)(ex_in + m * L::T) + (uint32_t)t * 4u)));
        } else {
            load_line<N>(x, buf_rsrc((const float2*)in + first, L::LPW * N * 8u), off * 8u);
        }
    } else {
#pragma unroll
        for (int m = 0; m < E; ++m) x[m] = make_float2(0.f, 0.f);
    }
    if constexpr (KIND == LK_FUSED) {
        float2 h[E];
        auto filter = [&] {
#pragma unroll
            for (int m = 0; m < E; ++m) h[m] = ld_off(H + m * L::T, (uint32_t)t * 8u);
        };
        if constexpr (OUT_H) {
            // twiddle reads one pass ahead where registers allow (forward from
            // 4096 points, inverse from 8192); from 8192 the inverse forms its
            // own products (kept ones would spill)
            if constexpr (N >= 4096) tw_first::fft_line_ahead<N, false>(x, lds, tw, t, filter);
            else tw_first::fft_line<N, false>(x, lds, tw, t, filter);
#pragma unroll
            for (int m = 0; m < E; ++m) x[m] = c_mul(x[m], h[m]);
            int ti = t;
            if constexpr (N >= 8192) asm volatile("" : "+v"(ti));
            if constexpr (N >= 8192) tw_first::fft_line_ahead<N, true>(x, lds, tw, ti);
            else tw_first::fft_line<N, true>(x, lds, tw, ti);
        } else {
            line_transform<N, LK_FUSED, PREC_FP32, true>(x, lds, H, tw, 1.0f, sub, t);
        }
    } else {
        static_assert(KIND == LK_FWD && OUT_H, "fused or forward");
        tw_first::fft_line_ahead<N, false>(x, lds, tw, t);
    }
    if constexpr (OUT_H) {
        const int e = half_exponent(line_absmax<N>(x, (float*)smem, sub));
        const float sc = ldexpf(1.0f, -e);
        if (live) {
            h2_t* dst = (h2_t*)out + first;
#pragma unroll
            for (int m = 0; m < E; ++m) {
                h2_t v;
                v.x = (_Float16)(x[m].x * sc);
                v.y = (_Float16)(x[m].y * sc);
                *(h2_t*)((char*)(dst + m * L::T) + off * 4u) = v;
            }
            if (t == 0) ex_out[line] = e;
        }
    } else if (live) {
        store_line<N>(x, buf_rsrc((float2*)out + first, L::LPW * N * 8u), off * 8u);
    }
}
#endif  // SAR_PART == 4

// ===================================================== launchers
static RcmcArgs make_rcmc_args(const RcmcHost& rh)
{
    RcmcArgs ra{};
    ra.stretch = rh.stretch;
    ra.rate = rh.rate;
    ra.table = rh.table;
    ra.r_near = rh.r_near;
    ra.stretch_max = rh.stretch_max;
    ra.x_per_bin = rh.x_per_bin;
    ra.two_over_lam = rh.two_over_lam;
    ra.nr = rh.nr;
    return ra;
}

constexpr int CUS = 256;                          // MI355X: 8 XCDs of 32 CUs

[[maybe_unused]] static int grid_for(long long work, int per_block)
{
    long long g = (work + per_block - 1) / per_block;
    const long long cap = CUS * 64LL;   // grid-stride kernels: 64 workgroups per CU
    return (int)(g < 1 ? 1 : (g > cap ? cap : g));
}

template <int N, int PREC>
static hipError_t set_lds_limit()
{
    using L = LineLaunch<N>;
    if (L::LDS_BYTES <= 64 * 1024) return hipSuccess;
    const void* fns[] = {(const void*)k_line<N, LK_FUSED, PREC, true>,
                         (const void*)k_line<N, LK_FWD, PREC, true>,
                         (const void*)k_line<N, LK_INV, PREC, true>,
                         (const void*)k_line<N, LK_FUSED, PREC, false>,
                         (const void*)k_line<N, LK_FWD, PREC, false>,
                         (const void*)k_line<N, LK_INV, PREC, false>,
                         (const void*)k_rcmc_az<N, 0, PREC>, (const void*)k_rcmc_az<N, 8, PREC>,
                         (const void*)k_rcmc_az2<N, PREC>,
                         (const void*)k_line_batch<N, LK_FUSED, PREC, true, true>,
                         (const void*)k_line_batch<N, LK_FWD, PREC, true, true>,
                         (const void*)k_line_batch<N, LK_INV, PREC, true, true>,
                         (const void*)k_line_batch<N, LK_FUSED, PREC, false, true>,
                         (const void*)k_line_batch<N, LK_FWD, PREC, false, true>,
                         (const void*)k_line_batch<N, LK_INV, PREC, false, true>,
                         (const void*)k_line_batch<N, LK_FUSED, PREC, true, false>,
                         (const void*)k_line_batch<N, LK_FWD, PREC, true, false>,
                         (const void*)k_line_batch<N, LK_INV, PREC, true, false>,
                         (const void*)k_line_batch<N, LK_FUSED, PREC, false, false>,
                         (const void*)k_line_batch<N, LK_FWD, PREC, false, false>,
                         (const void*)k_line_batch<N, LK_INV, PREC, false, false>};
    for (const void* f : fns) {
        const hipError_t e =
            hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS_BYTES);
        if (e != hipSuccess) return e;
    }
    if constexpr (PREC == PREC_FP32) {
        const void* split[] = {(const void*)k_line<N, LK_FWD, PREC, true, true>,
                               (const void*)k_line<N, LK_FWD, PREC, false, true>,
                               (const void*)k_line<N, LK_INV, PREC, true, true>,
                               (const void*)k_line<N, LK_INV, PREC, false, true>};
        for (const void* f : split) {
            const hipError_t e =
                hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS_BYTES);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

// FP32 line kernel with X times the default lines per workgroup.
template <int N, int KIND, bool TWP, bool SPLIT, int X>
static hipError_t launch_k_line_x(const float2* in, float2* out, int lines, const float2* H,
                                  const float2* tw, float scale, hipStream_t s)
{
    using L = LineLaunch<N, X>;
    static const hipError_t attr =
        L::LDS_BYTES <= 64 * 1024
            ? hipSuccess
            : hipFuncSetAttribute((const void*)k_line<N, KIND, PREC_FP32, TWP, SPLIT, X>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    const int groups = (lines + L::LPW - 1) / L::LPW;
    if (groups == 0) return hipSuccess;
    SAR_LAUNCH((k_line<N, KIND, PREC_FP32, TWP, SPLIT, X>), dim3(groups), dim3(L::BLOCK),
               L::LDS_BYTES, s, in, out, lines, H, tw, scale);
    return hipGetLastError();
}

// The persistent kernel is used for fused lines of 8192 points and more and
// single transforms of 16384 (the others run near the copy rate with one line
// per workgroup: 8192-point forward 182 us per 64 Mpx against 197, 4096-point
// fused inside a 4096^2 scene 205.7 us against 207.8 for the scene), once there
// are more lines than resident workgroups (below that there is no next line to
// load: 64 lines of 16384 take 16.2 us with k_line, 18.4 with it).
template <int N> constexpr int pipe_resident() { return CUS * (16384 / N); }
template <int N> static bool pipe_pays(int lines) { return lines > pipe_resident<N>(); }

template <int N, int KIND, bool TILED>
static hipError_t launch_pipe(const float2* in, float2* out, int lines, const float2* H,
                              const float2* tw, float scale, TileMap tm, hipStream_t s)
{
    using L = LineLaunch<N>;
    static const hipError_t attr =
        hipFuncSetAttribute((const void*)k_line_pipe<N, KIND, TILED>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    const int rounds = (lines + pipe_resident<N>() - 1) / pipe_resident<N>();
    const int grid = (lines + rounds - 1) / rounds;
    SAR_LAUNCH((k_line_pipe<N, KIND, TILED>), dim3(grid), dim3(L::BLOCK), L::LDS_BYTES, s, in, out,
               lines, H, tw, scale, tm);
    return hipGetLastError();
}

template <int N, int KIND, int PREC>
static hipError_t launch_k_line(const float2* in, float2* out, int lines, const float2* H,
                                const float2* tw, float scale, int variant, hipStream_t s)
{
    using L = LineLaunch<N>;
    const int groups = (lines + L::LPW - 1) / L::LPW;
    if (groups == 0) return hipSuccess;
    // variant bit 0: twiddles from the table (FP32 butterflies only); bit 1
    // (FP32 forward / inverse): the split real/imaginary exchange layout;
    // bit 2 (FP32, N <= 8192): twice the lines per workgroup
    if constexpr (PREC == PREC_FP32 && N <= 8192) {
        if (variant & 4) {
            const bool tab = variant & 1;
            if constexpr (KIND != LK_FUSED) {
                if (variant & 2)
                    return tab ? launch_k_line_x<N, KIND, false, true, 2>(in, out, lines, H, tw, scale, s)
                               : launch_k_line_x<N, KIND, true, true, 2>(in, out, lines, H, tw, scale, s);
            }
            return tab ? launch_k_line_x<N, KIND, false, false, 2>(in, out, lines, H, tw, scale, s)
                       : launch_k_line_x<N, KIND, true, false, 2>(in, out, lines, H, tw, scale, s);
        }
    }
    if constexpr (PREC == PREC_FP32 && (N == 16384 || (N == 8192 && KIND == LK_FUSED))) {
        if (variant == 0 && pipe_pays<N>(lines))
            return launch_pipe<N, KIND, false>(in, out, lines, H, tw, scale, TileMap{}, s);
    }
    if constexpr (PREC == PREC_FP32 && KIND != LK_FUSED) {
        if (variant & 2) {
            if (variant & 1)
                SAR_LAUNCH((k_line<N, KIND, PREC, false, true>), dim3(groups), dim3(L::BLOCK),
                                   L::LDS_BYTES, s, in, out, lines, H, tw, scale);
            else
                SAR_LAUNCH((k_line<N, KIND, PREC, true, true>), dim3(groups), dim3(L::BLOCK),
                                   L::LDS_BYTES, s, in, out, lines, H, tw, scale);
            return hipGetLastError();
        }
    }
    const bool keep = split_may_keep<N, KIND, PREC>() && groups <= 3 * CUS;
    if ((PREC == PREC_FP32 && (variant & 1)) || keep)
        SAR_LAUNCH((k_line<N, KIND, PREC, false>), dim3(groups), dim3(L::BLOCK),
                           L::LDS_BYTES, s, in, out, lines, H, tw, scale);
    else
        SAR_LAUNCH((k_line<N, KIND, PREC, true>), dim3(groups), dim3(L::BLOCK),
                           L::LDS_BYTES, s, in, out, lines, H, tw, scale);
    return hipGetLastError();
}

// k_rcmc_rows takes whole groups of rows and a shift that changes little per row.
template <int N> static bool rcmc_rows_fit(const RcmcArgs& ra)
{
    return ra.stretch_max <= RCMC_ROWS_STRETCH_MAX && ra.nr % (RcmcRows<N>::R * RcmcRows<N>::G) == 0;
}
template <int N, bool HIN, int PREC = PREC_FP32> static hipError_t allow_rcmc_rows_lds()
{
    return hipFuncSetAttribute((const void*)k_rcmc_rows<N, HIN, PREC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               RcmcRows<N>::LDS_BYTES);
}

template <int N, int PREC>
static hipError_t launch_line_n(LineOp op, const float2* in, float2* out, int lines,
                                const float2* H, const float2* tw, float scale,
                                const RcmcArgs* ra, int taps, int variant, hipStream_t s)
{
    using L = LineLaunch<N>;
    static const hipError_t attr = set_lds_limit<N, PREC>();
    if (attr != hipSuccess) return attr;
    switch (op) {
    case LineOp::Fused:
        return launch_k_line<N, LK_FUSED, PREC>(in, out, lines, H, tw, 1.0f, variant, s);
    case LineOp::Forward:
        return launch_k_line<N, LK_FWD, PREC>(in, out, lines, nullptr, tw, scale, variant, s);
    case LineOp::Inverse:
        return launch_k_line<N, LK_INV, PREC>(in, out, lines, nullptr, tw, scale, variant, s);
    case LineOp::RcmcAz: {
        const int groups = (lines + L::LPW - 1) / L::LPW;
        if (groups == 0) return hipSuccess;
        static_assert(L::LDS_BYTES >= RCMC_LDS_FLOATS * (int)sizeof(float), "table fits the line LDS");
        // variant bit 1: one output row per line slot instead of two; bit 2
        // (FP32, N = 4096 or 8192): the two rows on two line slots' threads
        // (k_rcmc_az2w) instead of one's
        const bool two_rows = taps == 8 && ra->stretch_max < 0.5 && (lines & 1) == 0 && !(variant & 2);
        if constexpr (PREC == PREC_FP32 && (N == 4096 || N == 8192)) {
            if (two_rows && (variant & 4)) {
                constexpr int lds2 = 2 * LineGeom<N>::LDS * (int)sizeof(float2);
                static const hipError_t wa =
                    lds2 <= 64 * 1024 ? hipSuccess
                                      : hipFuncSetAttribute((const void*)k_rcmc_az2w<N>,
                                                            hipFuncAttributeMaxDynamicSharedMemorySize,
                                                            lds2);
                if (wa != hipSuccess) return wa;
                SAR_LAUNCH((k_rcmc_az2w<N>), dim3(lines / 2), dim3(2 * LineGeom<N>::T), lds2,
                                   s, in, out, *ra, tw);
                return hipGetLastError();
            }
        }
        // four rows at a time where the geometry allows; at 16384 points one line
        // takes a CU's LDS and the two-row kernel was faster (208 us against 218
        // per 32 Mpx for two rows in two rounds).  Split butterflies alike: 4096^2
        // 101 -> 81 us, 1024^2 scene 48.0 -> 37.7, 128 x 512 39.6 -> 23.5
        if constexpr (N <= 8192) {
            if (two_rows && !(variant & 4) && rcmc_rows_fit<N>(*ra)) {
                static const hipError_t ga = allow_rcmc_rows_lds<N, false, PREC>();
                if (ga != hipSuccess) return ga;
                using Q = RcmcRows<N>;
                SAR_LAUNCH((k_rcmc_rows<N, false, PREC>), dim3(lines / (Q::R * Q::G)), dim3(Q::BLOCK),
                           Q::LDS_BYTES, s, in, out, *ra, tw);
                return hipGetLastError();
            }
        }
        if (two_rows) {
            const int g2 = (lines / 2 + L::LPW - 1) / L::LPW;
            SAR_LAUNCH((k_rcmc_az2<N, PREC>), dim3(g2), dim3(L::BLOCK), L::LDS_BYTES, s, in,
                               out, *ra, tw);
        } else if (taps == 8)
            SAR_LAUNCH((k_rcmc_az<N, 8, PREC>), dim3(groups), dim3(L::BLOCK), L::LDS_BYTES,
                               s, in, out, *ra, tw);
        else
            SAR_LAUNCH((k_rcmc_az<N, 0, PREC>), dim3(groups), dim3(L::BLOCK), L::LDS_BYTES,
                               s, in, out, *ra, tw);
        return hipGetLastError();
    }
    }
    return hipErrorInvalidValue;
}

template <int N, int PREC, bool TWP, bool PERSIST>
static void launch_line_batch_k(int kind, int grid, const LineTask* tasks, int ntasks,
                                int total_groups, float scale, hipStream_t s)
{
    using L = LineLaunch<N>;
    switch (kind) {
    case LK_FUSED:
        SAR_LAUNCH((k_line_batch<N, LK_FUSED, PREC, TWP, PERSIST>), dim3(grid),
                           dim3(L::BLOCK), L::LDS_BYTES, s, tasks, ntasks, total_groups, scale);
        break;
    case LK_FWD:
        SAR_LAUNCH((k_line_batch<N, LK_FWD, PREC, TWP, PERSIST>), dim3(grid),
                           dim3(L::BLOCK), L::LDS_BYTES, s, tasks, ntasks, total_groups, scale);
        break;
    default:
        SAR_LAUNCH((k_line_batch<N, LK_INV, PREC, TWP, PERSIST>), dim3(grid),
                           dim3(L::BLOCK), L::LDS_BYTES, s, tasks, ntasks, total_groups, scale);
        break;
    }
}

template <int N, int PREC, bool TWP>
static hipError_t launch_line_batch_t(int kind, const LineTask* tasks, int ntasks, int total_groups,
                                      float scale, int grid_sel, hipStream_t s)
{
    using L = LineLaunch<N>;
    static const hipError_t attr = set_lds_limit<N, PREC>();
    if (attr != hipSuccess) return attr;
    if (total_groups == 0) return hipSuccess;
    // grid_sel 0: one workgroup per line group; 1, 2, 3: a persistent grid of
    // 1x, 2x, 4x the resident workgroups (LDS-limited per CU x CUs)
    if ((grid_sel & 3) == 0) {
        launch_line_batch_k<N, PREC, TWP, false>(kind, total_groups, tasks, ntasks, total_groups,
                                                 scale, s);
        return hipGetLastError();
    }
    const int per_cu = (160 * 1024) / L::LDS_BYTES;
    const int resident = (per_cu < 1 ? 1 : per_cu) * CUS;
    const int cap = resident << ((grid_sel & 3) - 1);
    const int grid = total_groups < cap ? total_groups : cap;
    launch_line_batch_k<N, PREC, TWP, true>(kind, grid, tasks, ntasks, total_groups, scale, s);
    return hipGetLastError();
}

template <int N, int PREC>
static hipError_t launch_line_batch_n(int kind, const LineTask* tasks, int ntasks, int total_groups,
                                      float scale, int variant, hipStream_t s)
{
    // variant bit 0: table twiddles (FP32); bits 2-3: persistent grid size
    const int grid_sel = (variant >> 2) & 3;
    if (PREC == PREC_FP32 && (variant & 1))
        return launch_line_batch_t<N, PREC, false>(kind, tasks, ntasks, total_groups, scale,
                                                   grid_sel, s);
    return launch_line_batch_t<N, PREC, true>(kind, tasks, ntasks, total_groups, scale, grid_sel, s);
}

template <int PREC>
static hipError_t launch_line_batch_prec(int kind, int n, const LineTask* tasks, int ntasks,
                                         int total_groups, float scale, int v, hipStream_t s)
{
    switch (n) {
    case 64: return launch_line_batch_n<64, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 128: return launch_line_batch_n<128, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 256: return launch_line_batch_n<256, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 512: return launch_line_batch_n<512, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 1024: return launch_line_batch_n<1024, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 2048: return launch_line_batch_n<2048, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 4096: return launch_line_batch_n<4096, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 8192: return launch_line_batch_n<8192, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    case 16384: return launch_line_batch_n<16384, PREC>(kind, tasks, ntasks, total_groups, scale, v, s);
    default: return hipErrorInvalidValue;
    }
}

template <int PREC>
static hipError_t launch_line_prec(LineOp op, int n, const float2* i, float2* o, int lines,
                                   const float2* h, const float2* w, float scale,
                                   const RcmcArgs* ra, int taps, int v, hipStream_t s)
{
    switch (n) {
    case 64: return launch_line_n<64, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 128: return launch_line_n<128, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 256: return launch_line_n<256, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 512: return launch_line_n<512, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 1024: return launch_line_n<1024, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 2048: return launch_line_n<2048, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 4096: return launch_line_n<4096, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 8192: return launch_line_n<8192, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    case 16384: return launch_line_n<16384, PREC>(op, i, o, lines, h, w, scale, ra, taps, v, s);
    default: return hipErrorInvalidValue;
    }
}

// One instantiation of launch_line_prec / launch_line_batch_prec per part
// (defined in parts 1-3).
hipError_t launch_line_batch_p1(int, int, const LineTask*, int, int, float, int, hipStream_t);
hipError_t launch_line_batch_p2(int, int, const LineTask*, int, int, float, int, hipStream_t);
hipError_t launch_line_batch_p3(int, int, const LineTask*, int, int, float, int, hipStream_t);
hipError_t launch_line_fp32(LineOp, int, const float2*, float2*, int, const float2*, const float2*,
                            float, const RcmcArgs*, int, int, hipStream_t);
hipError_t launch_line_f16(LineOp, int, const float2*, float2*, int, const float2*, const float2*,
                           float, const RcmcArgs*, int, int, hipStream_t);
hipError_t launch_line_bf16(LineOp, int, const float2*, float2*, int, const float2*, const float2*,
                            float, const RcmcArgs*, int, int, hipStream_t);

#if SAR_PART >= 1 && SAR_PART <= 3
hipError_t SAR_LINE_BATCH_FN(int kind, int n, const LineTask* tasks, int ntasks, int total_groups,
                             float scale, int v, hipStream_t s)
{
    return launch_line_batch_prec<SAR_PART - 1>(kind, n, tasks, ntasks, total_groups, scale, v, s);
}
#endif

#if SAR_PART == 1
hipError_t launch_line_fp32(LineOp op, int n, const float2* i, float2* o, int lines,
                            const float2* h, const float2* w, float scale, const RcmcArgs* ra,
                            int taps, int v, hipStream_t s)
{
    return launch_line_prec<PREC_FP32>(op, n, i, o, lines, h, w, scale, ra, taps, v, s);
}
#elif SAR_PART == 4

template <int N>
static hipError_t launch_range_tiled_n(const float2* in, float2* out, int na, const float2* H,
                                       const float2* tw, hipStream_t s)
{
    using L = LineLaunch<N>;
    const TileMap tm = tile_map(na);
    if constexpr (N >= 8192) {
        if (pipe_pays<N>(na)) return launch_pipe<N, LK_FUSED, true>(in, out, na, H, tw, 1.0f, tm, s);
    }
    static const hipError_t attr =
        L::LDS_BYTES <= 64 * 1024
            ? hipSuccess
            : hipFuncSetAttribute((const void*)k_line_tiled<N>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    SAR_LAUNCH((k_line_tiled<N>), dim3(na / L::LPW), dim3(L::BLOCK), L::LDS_BYTES, s, in, out, H, tw, tm);
    return hipGetLastError();
}

hipError_t launch_range_tiled(int n, const void* in, void* out, int na, const void* H, const void* tw,
                              hipStream_t s)
{
    if (na < 64 || (na & 63) != 0) return hipErrorInvalidValue;   // whole workgroups and tiles
    auto i = (const float2*)in;
    auto o = (float2*)out;
    auto h = (const float2*)H;
    auto w = (const float2*)tw;
    switch (n) {
    case 64: return launch_range_tiled_n<64>(i, o, na, h, w, s);
    case 128: return launch_range_tiled_n<128>(i, o, na, h, w, s);
    case 256: return launch_range_tiled_n<256>(i, o, na, h, w, s);
    case 512: return launch_range_tiled_n<512>(i, o, na, h, w, s);
    case 1024: return launch_range_tiled_n<1024>(i, o, na, h, w, s);
    case 2048: return launch_range_tiled_n<2048>(i, o, na, h, w, s);
    case 4096: return launch_range_tiled_n<4096>(i, o, na, h, w, s);
    case 8192: return launch_range_tiled_n<8192>(i, o, na, h, w, s);
    case 16384: return launch_range_tiled_n<16384>(i, o, na, h, w, s);
    default: return hipErrorInvalidValue;
    }
}

template <int N, int KIND, int CW, bool BACK = false>
static hipError_t launch_strip_k(const float2* in, float2* out, int cols, const float2* H,
                                 const float2* tw, float scale, hipStream_t s)
{
    using S = StripLaunch<N, CW>;
    static const hipError_t attr =
        S::LDS_BYTES <= 64 * 1024
            ? hipSuccess
            : hipFuncSetAttribute((const void*)k_line_strip<N, KIND, CW, BACK>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    // whole strips and tiles; 16-byte pair loads need an aligned base
    if (cols % TILE_COLS != 0 || ((uintptr_t)in & 15u)) return hipErrorInvalidValue;
    if (cols == 0) return hipSuccess;
    SAR_LAUNCH((k_line_strip<N, KIND, CW, BACK>), dim3(cols / S::C), dim3(S::BLOCK), S::LDS_BYTES,
               s, in, out, cols, tile_map(N), H, tw, scale);
    return hipGetLastError();
}

template <int N, int CW>
static hipError_t launch_strip_c(StripOp op, const float2* in, float2* out, int cols, const float2* H,
                                 const float2* tw, float scale, hipStream_t s)
{
    switch (op) {
    case StripOp::Fused: return launch_strip_k<N, LK_FUSED, CW>(in, out, cols, H, tw, 1.f, s);
    case StripOp::FusedBack: return launch_strip_k<N, LK_FUSED, CW, true>(in, out, cols, H, tw, 1.f, s);
    case StripOp::Forward: return launch_strip_k<N, LK_FWD, CW>(in, out, cols, nullptr, tw, scale, s);
    }
    return hipErrorInvalidValue;
}

// The strip width is the default one where that makes a workgroup per CU, else half
// of it, else the narrowest of whole waves (two lines from 512 points): with few
// range cells the chip would stand idle (2048 x 256 scene: 24.0 us with 32 strips of
// 8, 17.4 with 128 of 2).  Variant 1, tuned per line length whatever the number of
// range cells: half in place of the default width, not in place of a narrower one.
template <int N>
static hipError_t launch_strip_n(StripOp op, const float2* in, float2* out, int cols,
                                 const float2* H, const float2* tw, float scale, int variant,
                                 hipStream_t s)
{
    constexpr int C = StripLaunch<N>::C_DEFAULT, HALF = C / 2;
    constexpr int LEAST = 64 / StripLaunch<N>::T > 2 ? 64 / StripLaunch<N>::T : 2;
    if constexpr (LEAST < HALF) {
        if (cols / HALF < CUS) return launch_strip_c<N, LEAST>(op, in, out, cols, H, tw, scale, s);
    }
    if constexpr (LEAST <= HALF) {
        if (cols / C < CUS) return launch_strip_c<N, HALF>(op, in, out, cols, H, tw, scale, s);
    }
    if (variant == 1) return launch_strip_c<N, HALF>(op, in, out, cols, H, tw, scale, s);
    return launch_strip_c<N, C>(op, in, out, cols, H, tw, scale, s);
}

bool strip_width_open(int n, int cols)
{
    switch (n) {
#define SAR_CASE(N) case N: return StripLaunch<N>::T < 8 || cols / StripLaunch<N>::C_DEFAULT >= CUS;
        SAR_CASE(64) SAR_CASE(128) SAR_CASE(256) SAR_CASE(512) SAR_CASE(1024) SAR_CASE(2048) SAR_CASE(4096)
#undef SAR_CASE
    default: return false;
    }
}

hipError_t launch_line_strip(StripOp op, int n, const void* in, void* out, int cols,
                             const void* H, const void* tw, float scale, int variant, hipStream_t s)
{
    auto i = (const float2*)in;
    auto o = (float2*)out;
    auto h = (const float2*)H;
    auto w = (const float2*)tw;
    switch (n) {
    case 64: return launch_strip_n<64>(op, i, o, cols, h, w, scale, variant, s);
    case 128: return launch_strip_n<128>(op, i, o, cols, h, w, scale, variant, s);
    case 256: return launch_strip_n<256>(op, i, o, cols, h, w, scale, variant, s);
    case 512: return launch_strip_n<512>(op, i, o, cols, h, w, scale, variant, s);
    case 1024: return launch_strip_n<1024>(op, i, o, cols, h, w, scale, variant, s);
    case 2048: return launch_strip_n<2048>(op, i, o, cols, h, w, scale, variant, s);
    case 4096: return launch_strip_n<4096>(op, i, o, cols, h, w, scale, variant, s);
    default: return hipErrorInvalidValue;
    }
}

int batch_range_groups(int n, int lines)
{
    const int lpw = BATCH_RANGE_BLOCK * 16 / n;
    return (lines + lpw - 1) / lpw;
}

int batch_strip_groups(int n, int lines)
{
    switch (n) {
#define SAR_CASE(N) case N: return lines / (BatchStrip<N>::C * BatchStrip<N>::PER_WG);
        SAR_BATCH_LENGTHS(SAR_CASE)
#undef SAR_CASE
    default: return 0;
    }
}

hipError_t launch_batch_range(const void* tasks, int ntasks, int total, hipStream_t s)
{
    static_assert(BATCH_RANGE_LDS <= 64 * 1024, "needs no LDS attribute");
    if (total == 0) return hipSuccess;
    SAR_LAUNCH(k_batch_range, dim3(total), dim3(BATCH_RANGE_BLOCK), BATCH_RANGE_LDS, s,
               (const SceneTask*)tasks, ntasks);
    return hipGetLastError();
}

hipError_t launch_batch_strip(const void* tasks, int ntasks, int total, hipStream_t s)
{
    static_assert(BATCH_STRIP_LDS <= 64 * 1024, "needs no LDS attribute");
    if (total == 0) return hipSuccess;
    SAR_LAUNCH(k_batch_strip, dim3(total), dim3(BATCH_STRIP_BLOCK), BATCH_STRIP_LDS, s,
               (const SceneTask*)tasks, ntasks, total);
    return hipGetLastError();
}

template <const void* (*KERNEL)(), int BYTES>
static hipError_t allow_lds()
{
    static const hipError_t e =
        BYTES <= 64 * 1024
            ? hipSuccess
            : hipFuncSetAttribute(KERNEL(), hipFuncAttributeMaxDynamicSharedMemorySize, BYTES);
    return e;
}

template <int N, int KIND, bool IN_H, bool OUT_H>
static const void* hs_kernel() { return (const void*)k_line_hs<N, KIND, IN_H, OUT_H>; }

template <int N, int KIND, bool IN_H, bool OUT_H>
static hipError_t launch_hs_n(const void* in, void* out, int lines, const void* H, const void* tw,
                              const int* ex_in, int* ex_out, hipStream_t s)
{
    using L = LineLaunch<N>;
    const hipError_t attr = allow_lds<hs_kernel<N, KIND, IN_H, OUT_H>, L::LDS_BYTES>();
    if (attr != hipSuccess) return attr;
    const int groups = (lines + L::LPW - 1) / L::LPW;
    if (groups == 0) return hipSuccess;
    SAR_LAUNCH((k_line_hs<N, KIND, IN_H, OUT_H>), dim3(groups), dim3(L::BLOCK),
                       L::LDS_BYTES, s, in, out, lines, (const float2*)H, (const float2*)tw, ex_in,
                       ex_out);
    return hipGetLastError();
}

template <int N>
static hipError_t launch_hs_op(HalfOp op, const void* in, void* out, int lines, const void* H,
                               const void* tw, const int* ex_in, int* ex_out, hipStream_t s)
{
    switch (op) {
    case HalfOp::RangeFused:
        return launch_hs_n<N, LK_FUSED, false, true>(in, out, lines, H, tw, ex_in, ex_out, s);
    case HalfOp::AzimuthFused:
        return launch_hs_n<N, LK_FUSED, true, false>(in, out, lines, H, tw, ex_in, ex_out, s);
    case HalfOp::AzimuthForward:
        return launch_hs_n<N, LK_FWD, true, true>(in, out, lines, H, tw, ex_in, ex_out, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_line_half(HalfOp op, int n, const void* in, void* out, int lines, const void* H,
                            const void* tw, const int* ex_in, int* ex_out, hipStream_t s)
{
    switch (n) {
    case 64: return launch_hs_op<64>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 128: return launch_hs_op<128>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 256: return launch_hs_op<256>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 512: return launch_hs_op<512>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 1024: return launch_hs_op<1024>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 2048: return launch_hs_op<2048>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 4096: return launch_hs_op<4096>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 8192: return launch_hs_op<8192>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    case 16384: return launch_hs_op<16384>(op, in, out, lines, H, tw, ex_in, ex_out, s);
    default: return hipErrorInvalidValue;
    }
}

template <int N>
static const void* rcmc_half_kernel() { return (const void*)k_rcmc_az2<N, PREC_FP32, true>; }

template <int N>
static hipError_t launch_rcmc_half_n(const void* A, const int* ex, void* out, const RcmcArgs& ra0,
                                     const void* tw, hipStream_t s)
{
    using L = LineLaunch<N>;
    const hipError_t attr = allow_lds<rcmc_half_kernel<N>, L::LDS_BYTES>();
    if (attr != hipSuccess) return attr;
    RcmcArgs ra = ra0;
    ra.row_exp = ex;
    if constexpr (N <= 8192) {
        if (rcmc_rows_fit<N>(ra)) {
            static const hipError_t ga = allow_rcmc_rows_lds<N, true>();
            if (ga != hipSuccess) return ga;
            using Q = RcmcRows<N>;
            SAR_LAUNCH((k_rcmc_rows<N, true>), dim3(ra.nr / (Q::R * Q::G)), dim3(Q::BLOCK), Q::LDS_BYTES, s,
                       A, (float2*)out, ra, (const float2*)tw);
            return hipGetLastError();
        }
    }
    const int g2 = (ra.nr / 2 + L::LPW - 1) / L::LPW;
    if (g2 == 0) return hipSuccess;
    SAR_LAUNCH((k_rcmc_az2<N, PREC_FP32, true>), dim3(g2), dim3(L::BLOCK), L::LDS_BYTES, s,
                       A, (float2*)out, ra, (const float2*)tw);
    return hipGetLastError();
}

hipError_t launch_rcmc_half(int n, const void* A, const int* ex, void* out, const RcmcHost& rh,
                            const void* tw, hipStream_t s)
{
    if (rh.taps != 8 || !(rh.stretch_max < 0.5) || (rh.nr & 1)) return hipErrorInvalidValue;
    const RcmcArgs ra = make_rcmc_args(rh);
    switch (n) {
    case 64: return launch_rcmc_half_n<64>(A, ex, out, ra, tw, s);
    case 128: return launch_rcmc_half_n<128>(A, ex, out, ra, tw, s);
    case 256: return launch_rcmc_half_n<256>(A, ex, out, ra, tw, s);
    case 512: return launch_rcmc_half_n<512>(A, ex, out, ra, tw, s);
    case 1024: return launch_rcmc_half_n<1024>(A, ex, out, ra, tw, s);
    case 2048: return launch_rcmc_half_n<2048>(A, ex, out, ra, tw, s);
    case 4096: return launch_rcmc_half_n<4096>(A, ex, out, ra, tw, s);
    case 8192: return launch_rcmc_half_n<8192>(A, ex, out, ra, tw, s);
    case 16384: return launch_rcmc_half_n<16384>(A, ex, out, ra, tw, s);
    default: return hipErrorInvalidValue;
    }
}
#elif SAR_PART == 2
hipError_t launch_line_f16(LineOp op, int n, const float2* i, float2* o, int lines,
                           const float2* h, const float2* w, float scale, const RcmcArgs* ra,
                           int taps, int v, hipStream_t s)
{
    return launch_line_prec<PREC_F16>(op, n, i, o, lines, h, w, scale, ra, taps, v, s);
}
#elif SAR_PART == 3
hipError_t launch_line_bf16(LineOp op, int n, const float2* i, float2* o, int lines,
                            const float2* h, const float2* w, float scale, const RcmcArgs* ra,
                            int taps, int v, hipStream_t s)
{
    return launch_line_prec<PREC_BF16>(op, n, i, o, lines, h, w, scale, ra, taps, v, s);
}
#endif

#if SAR_PART == 0
hipError_t launch_line(LineOp op, int n, const void* in, void* out, int lines, const void* H,
                       const void* tw, float scale, const RcmcHost* rh, int prec, int variant,
                       hipStream_t s)
{
    RcmcArgs ra{};
    int taps = 0;
    if (rh) {
        ra = make_rcmc_args(*rh);
        taps = rh->taps;
    }
    auto i = (const float2*)in;
    auto o = (float2*)out;
    auto h = (const float2*)H;
    auto w = (const float2*)tw;
    switch (prec) {
    case PREC_FP32: return launch_line_fp32(op, n, i, o, lines, h, w, scale, &ra, taps, variant, s);
    case PREC_F16: return launch_line_f16(op, n, i, o, lines, h, w, scale, &ra, taps, variant, s);
    case PREC_BF16: return launch_line_bf16(op, n, i, o, lines, h, w, scale, &ra, taps, variant, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_line_batch(int kind, int n, const void* tasks, int ntasks, int total_groups,
                             float scale, int prec, int variant, hipStream_t s)
{
    const LineTask* t = (const LineTask*)tasks;
    switch (prec) {
    case PREC_FP32: return launch_line_batch_p1(kind, n, t, ntasks, total_groups, scale, variant, s);
    case PREC_F16: return launch_line_batch_p2(kind, n, t, ntasks, total_groups, scale, variant, s);
    case PREC_BF16: return launch_line_batch_p3(kind, n, t, ntasks, total_groups, scale, variant, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_corner_turn_batch(const void* tasks, int ntasks, int total_tiles, hipStream_t s)
{
    if (total_tiles == 0) return hipSuccess;
    const int grid = total_tiles < CUS * 16 ? total_tiles : CUS * 16;
    SAR_LAUNCH(k_corner_turn_batch, dim3(grid), dim3(256), 0, s, (const TurnTask*)tasks,
                       ntasks, total_tiles);
    return hipGetLastError();
}

int line_groups(int n, int lines)
{
    const int T = n / line_e(n);
    const int lpw = T >= 256 ? 1 : 256 / T;
    return (lines + lpw - 1) / lpw;
}

int turn_tiles(int rows, int cols) { return ((rows + TT - 1) / TT) * ((cols + TT - 1) / TT); }

int twiddle_table_size(int n)
{
    switch (n) {
    case 64: return LineGeom<64>::TW_SIZE;
    case 128: return LineGeom<128>::TW_SIZE;
    case 256: return LineGeom<256>::TW_SIZE;
    case 512: return LineGeom<512>::TW_SIZE;
    case 1024: return LineGeom<1024>::TW_SIZE;
    case 2048: return LineGeom<2048>::TW_SIZE;
    case 4096: return LineGeom<4096>::TW_SIZE;
    case 8192: return LineGeom<8192>::TW_SIZE;
    case 16384: return LineGeom<16384>::TW_SIZE;
    default: return -1;
    }
}

hipError_t launch_rowmul(const void* in, void* out, int rows, int n, const void* H, hipStream_t s)
{
    const long long pairs = (long long)rows * n / 2;
    SAR_LAUNCH(k_rowmul, dim3(grid_for(pairs, 256)), dim3(256), 0, s, (const float4*)in,
                       (float4*)out, pairs, n, (const float2*)H);
    return hipGetLastError();
}

hipError_t launch_corner_turn_b4(const void* in, void* out, int rows, int cols, hipStream_t s)
{
    if (rows % TT != 0 || cols % TT != 0 || (((uintptr_t)in | (uintptr_t)out) & 7u) != 0)
        return hipErrorInvalidValue;
    const long long tiles = (long long)(rows / TT) * (cols / TT);
    if (tiles == 0) return hipSuccess;
    SAR_LAUNCH(k_corner_turn_b4, dim3((unsigned)tiles), dim3(256), 0, s, (const uint2*)in,
                       (uint2*)out, rows, cols);
    return hipGetLastError();
}

hipError_t launch_corner_turn(const void* in, void* out, int rows, int cols, int variant,
                              hipStream_t s)
{
    const long long tiles = (long long)((rows + TT - 1) / TT) * ((cols + TT - 1) / TT);
    if (tiles == 0) return hipSuccess;
    const bool whole = rows % TT == 0 && cols % TT == 0 &&
                       (((uintptr_t)in | (uintptr_t)out) & 15u) == 0;
    if (whole) {
        // a grid of at most 1280 workgroups (five per CU, as many as LDS
        // holds), each taking the same number of tiles (the last round
        // ragged); variant 1: at most 1024 (four per CU); variant 2: one
        // workgroup per tile.  The tiles and their order within a workgroup
        // do not change the result.
        const long long cap = variant == 1 ? 1024 : (variant == 2 ? tiles : 1280);
        const long long per = (tiles + cap - 1) / cap;
        const long long grid = (tiles + per - 1) / per;
        SAR_LAUNCH(k_corner_turn_x2, dim3((unsigned)grid), dim3(256), 0, s,
                           (const float4*)in, (float4*)out, rows, cols, (int)tiles);
    }
    // output rows that start on 64-byte boundaries: 64-row tiles (3000 x 5001:
    // 51.1 us against 52.5 with 128 rows, 1000 x 777: 4.3 against 5.0); others:
    // 128-row tiles (5001 x 3000: 57.5 against 62.0, 4097 x 4097: 60 against 64)
    else if (rows % 8 == 0 && ((uintptr_t)out & 63u) == 0)
        SAR_LAUNCH(k_corner_turn<64>, dim3((unsigned)tiles), dim3(256), 0, s, (const float2*)in,
                           (float2*)out, rows, cols);
    else {
        const long long tall = (long long)((rows + 127) / 128) * ((cols + TT - 1) / TT);
        SAR_LAUNCH(k_corner_turn<128>, dim3((unsigned)tall), dim3(512), 0, s, (const float2*)in,
                           (float2*)out, rows, cols);
    }
    return hipGetLastError();
}

hipError_t launch_rcmc_interp(const void* A, void* out, int na, const RcmcHost& rh, hipStream_t s)
{
    const RcmcArgs ra = make_rcmc_args(rh);
    const long long total = (long long)rh.nr * na;
    if (rh.taps == 8)
        SAR_LAUNCH(k_rcmc_interp<8>, dim3(grid_for(total, 256)), dim3(256), 0, s,
                           (const float2*)A, (float2*)out, na, ra);
    else
        SAR_LAUNCH(k_rcmc_interp<0>, dim3(grid_for(total, 256)), dim3(256), 0, s,
                           (const float2*)A, (float2*)out, na, ra);
    return hipGetLastError();
}

hipError_t launch_az_phase(const void* in, void* out, int na, const RcmcHost& rh, float scale,
                           hipStream_t s)
{
    const RcmcArgs ra = make_rcmc_args(rh);
    const long long total = (long long)rh.nr * na;
    SAR_LAUNCH(k_az_phase, dim3(grid_for(total, 256)), dim3(256), 0, s, (const float2*)in,
                       (float2*)out, na, ra, scale);
    return hipGetLastError();
}

hipError_t launch_gen_twiddles(void* tw, int n, hipStream_t s)
{
    const int cnt = twiddle_table_size(n);
    if (cnt <= 0) return hipSuccess;
    SAR_LAUNCH(k_gen_twiddles, dim3((cnt + 255) / 256), dim3(256), 0, s, (float2*)tw, n,
                       line_e(n));
    return hipGetLastError();
}

hipError_t launch_gen_chirp_filter(void* H, int n, int len, double K, int sign, double scale,
                                   hipStream_t s)
{
    SAR_LAUNCH(k_gen_chirp_filter, dim3((n + 255) / 256), dim3(256), 0, s, (float2*)H, n,
                       len, K, sign, scale);
    return hipGetLastError();
}

hipError_t launch_gen_rcmc_table(float* tab, double beta, hipStream_t s)
{
    static_assert(RROWS_INTERVALS <= RCMC_INTERVALS, "one thread per interval");
    SAR_LAUNCH(k_gen_rcmc_table, dim3(2), dim3(RCMC_INTERVALS), 0, s, tab, beta);
    return hipGetLastError();
}

int rcmc_table_floats() { return RCMC_TAB; }
int rcmc_all_floats() { return RCMC_TAB + RROWS_TAB; }

hipError_t launch_gen_hyper_tables(double* stretch, double* rate, int na, double lam, double v,
                                   hipStream_t s)
{
    // the same expressions as the kernels' RcmcArgs (x_per_bin, two_over_lam)
    SAR_LAUNCH(k_gen_hyper_tables, dim3((na + 255) / 256), dim3(256), 0, s, stretch, rate,
                       na, lam / (2.0 * v * (double)na), 2.0 / lam);
    return hipGetLastError();
}

#endif  // SAR_PART == 0

}  // namespace sar
