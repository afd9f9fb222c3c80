// Boxcar integration and S/N on gfx950.
//
// A dedispersed row is processed in LDS chunks.  Each chunk holds the
// exclusive prefix sum Q of `chunk` consecutive samples (uint32, modulo 2^32);
// a boxcar of width w starting at local index u is then Q[u + w] - Q[u],
// exact in int32 because the true sum fits (wrap-around cancels).  Chunks
// overlap by H >= max width samples so every output of a chunk finds its whole
// window inside it; all widths are served from the same prefix array.
//
// The prefix array lives in LDS unpadded.  Lane l of the prefix pass owns
// samples 16 l - 1 .. 16 l + 14 of the chunk (the first lane's first is
// zero), so its 16 prefix values are Q[16 l .. 16 l + 15], four aligned
// 16-byte stores.  The statistics read Q[u .. u + 3] and Q[u + w .. u + w + 3]
// (u a multiple of 4) as one aligned 16-byte load each when 4 divides w, and
// as dword loads at immediate offsets otherwise, so no per-element index
// arithmetic remains.  (A layout padded by 4 dwords per 64, or assembling
// widths 1 to 3 in registers from two aligned groups, measured slower.)
//
// S/N statistics per (width, row): per work-item the running maximum with its
// first index (strictly greater replaces it, and each work-item visits its
// outputs in increasing t), and FP64 sums of (x - r) and (x - r)^2 about an
// integer reference r close to the series mean.  For the reduction across
// wavefronts the maximum is packed as one int64 key (value << 32 | ~t) so
// that a plain max keeps the earliest peak; the finish is FP64.  Bounds are
// tested per element only in a work-item's last, partial step.
#include "internal.h"

#include <algorithm>
#include <cfloat>
#include <climits>
#include <type_traits>
#include <utility>

namespace amber {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));


// Widths of the sliding boxcars, or (dec != 0) decimation factors: then entry
// k is the series of sums of w[k] consecutive samples starting at multiples
// of w[k], i.e. the width-w[k] boxcar read at t = j w[k], j < n_out / w[k].
struct WidthSet {
    int32_t w[AMBER_MAX_WIDTHS];
    int32_t step[AMBER_MAX_WIDTHS];
    int32_t n;
    int32_t dec;
};

struct Stat {
    long long key;
    double s1, s2;
};

__device__ __forceinline__ long long pack_key(int32_t x, int64_t t)
{
    // high half: the signed value; low half: ~t, so equal values prefer the earlier t
    return (long long)(((uint64_t)(int64_t)x << 32) | (uint64_t)(0xffffffffu - (uint32_t)t));
}

__device__ __forceinline__ void stat_init(Stat &s)
{
    s.key = LLONG_MIN;
    s.s1 = 0.0;
    s.s2 = 0.0;
}

__device__ __forceinline__ void stat_add(Stat &s, int32_t x, int64_t t, double r)
{
    const long long k = pack_key(x, t);
    s.key = k > s.key ? k : s.key;
    const double d = (double)x - r;
    s.s1 += d;
    s.s2 = fma(d, d, s.s2);
}

// Running statistics of one work-item: values arrive in increasing t, so a
// strictly greater value is the only one that replaces the maximum.  Values
// are > INT32_MIN (|box| < 2^31 by the callers' contract).
struct Run {
    int32_t vmax;
    uint32_t tmax;
    double s1, s2;
};

__device__ __forceinline__ void run_init(Run &s)
{
    s.vmax = INT32_MIN;
    s.tmax = 0xffffffffu;
    s.s1 = 0.0;
    s.s2 = 0.0;
}

__device__ __forceinline__ void run_add(Run &s, int32_t x, uint32_t t, double r)
{
    const bool up = x > s.vmax;
    s.vmax = up ? x : s.vmax;
    s.tmax = up ? t : s.tmax;
    const double d = (double)x - r;
    s.s1 += d;
    s.s2 = fma(d, d, s.s2);
}

__device__ __forceinline__ Stat run_stat(const Run &s)
{
    Stat o;
    o.key = pack_key(s.vmax, s.tmax);  // the initial state packs to LLONG_MIN
    o.s1 = s.s1;
    o.s2 = s.s2;
    return o;
}

__device__ __forceinline__ Stat wave_reduce(Stat s)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const long long k = __shfl_xor(s.key, off, 64);
        s.key = k > s.key ? k : s.key;
        s.s1 += __shfl_xor(s.s1, off, 64);
        s.s2 += __shfl_xor(s.s2, off, 64);
    }
    return s;
}

// Writes (snr, peak) of one series of N values from its reduced statistics.
__device__ __forceinline__ void finish(const Stat &s, int64_t n, double r, float *snr, int32_t *peak)
{
    const int32_t vmax = (int32_t)(s.key >> 32);
    const uint32_t t = 0xffffffffu - (uint32_t)(s.key & 0xffffffffll);
    const double m1 = s.s1 / (double)n;
    double var = s.s2 / (double)n - m1 * m1;
    var = var > 0.0 ? var : 0.0;
    const double sigma = sqrt(var);
    const double excess = ((double)vmax - r) - m1;
    *snr = sigma > 0.0 ? (float)(excess / sigma) : 0.0f;
    if (peak) *peak = (int32_t)t;
}

// Block reduction of per-thread stats for NW widths; thread k < n_w receives
// width k's total.  scratch holds NW * 16 Stats.
template <int NW>
__device__ __forceinline__ void block_reduce(Stat (&st)[NW], int n_w, Stat *scratch)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        if (k < n_w) {
            Stat r = wave_reduce(st[k]);
            if (lane == 0) scratch[k * 16 + wave] = r;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < n_w) {
        const int k = threadIdx.x;
        Stat tot = scratch[k * 16];
        for (int w = 1; w < waves; ++w) {
            const Stat o = scratch[k * 16 + w];
            tot.key = o.key > tot.key ? o.key : tot.key;
            tot.s1 += o.s1;
            tot.s2 += o.s2;
        }
        scratch[k * 16] = tot;
    }
    __syncthreads();
}

// Loads samples [cs, cs + chunk) of one row (zero past n_out) and writes the
// exclusive prefix Q[0 .. chunk) to LDS.  Work-item l loads samples
// 16 l .. 16 l + 15 and takes sample 16 l - 1 from its left neighbour (zero
// for the first), so that its 16 prefix values are Q[16 l .. 16 l + 15].
__device__ __forceinline__ void load_prefix(const int32_t *__restrict__ row, int64_t cs, int64_t n_out, bool vec_ok,
                                            uint32_t *Q, uint32_t *wave_tot)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    const int64_t base = cs + (int64_t)tid * 16;
    uint32_t x[16];
    if (vec_ok && base + 16 <= n_out) {
        const int4 *p = reinterpret_cast<const int4 *>(row + base);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int4 v = p[q];
            x[4 * q + 0] = (uint32_t)v.x; x[4 * q + 1] = (uint32_t)v.y;
            x[4 * q + 2] = (uint32_t)v.z; x[4 * q + 3] = (uint32_t)v.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = (base + e < n_out) ? (uint32_t)row[base + e] : 0u;
    }
    // sample 16 l - 1: the left lane's last; a wave's first lane reads it
    uint32_t left = __shfl_up(x[15], 1, 64);
    if (lane == 0) left = (tid > 0 && base - 1 < n_out) ? (uint32_t)row[base - 1] : 0u;
    uint32_t v[16];
    v[0] = left;
#pragma unroll
    for (int e = 1; e < 16; ++e) v[e] = v[e - 1] + x[e - 1];
    // inclusive scan of work-item totals (samples 16 l - 1 .. 16 l + 14) within the wave
    uint32_t incl = v[15];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    if (tid == 0) {
        uint32_t run = 0;
        for (int w = 0; w < waves; ++w) {
            const uint32_t y = wave_tot[w];
            wave_tot[w] = run;
            run += y;
        }
    }
    __syncthreads();
    const uint32_t excl = incl - v[15] + wave_tot[wave];
    u32x4 *dst = reinterpret_cast<u32x4 *>(Q + tid * 16);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        dst[q] = u32x4{v[4 * q] + excl, v[4 * q + 1] + excl, v[4 * q + 2] + excl, v[4 * q + 3] + excl};
    __syncthreads();
}

// Loads Q[base .. base + S) (logical indices).  S >= 4 and base a multiple
// of 4: one aligned 16-byte load per group of four; otherwise dword loads.
template <int S>
__device__ __forceinline__ void load_q(const uint32_t *Q, int base, bool aligned, uint32_t (&v)[S])
{
    if (S >= 4 && aligned) {
#pragma unroll
        for (int q = 0; q < S / 4; ++q) {
            const u32x4 x = *reinterpret_cast<const u32x4 *>(Q + base + 4 * q);
            v[4 * q + 0] = x.x;
            v[4 * q + 1] = x.y;
            v[4 * q + 2] = x.z;
            v[4 * q + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int s = 0; s < S; ++s) v[s] = Q[base + s];
    }
}

// Accumulates width w over the chunk's outputs [cs, cs + outs) with S
// consecutive outputs per work-item per step.
template <int S>
__device__ __forceinline__ void width_stats(const uint32_t *Q, int w, int outs, int64_t cs, int64_t n_valid, double r,
                                            Run &st)
{
    const bool w_aligned = (w & 3) == 0;
    for (int g = threadIdx.x; g * S < outs; g += blockDim.x) {
        const int u = g * S;
        uint32_t a[S], b[S];
        load_q<S>(Q, u, true, a);
        load_q<S>(Q, u + w, w_aligned, b);
        const uint32_t t0 = (uint32_t)(cs + u);
        if (u + S <= outs && cs + u + S <= n_valid) {
#pragma unroll
            for (int s = 0; s < S; ++s) run_add(st, (int32_t)(b[s] - a[s]), t0 + s, r);
        } else {  // the last, partial step
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (u + s < outs && cs + u + s < n_valid) run_add(st, (int32_t)(b[s] - a[s]), t0 + s, r);
        }
    }
}

// Accumulates the decimated series of factor f over the bins j whose first
// sample j f lies in [cs, cs + outs), j < n_bins, S bins per work-item per step.
template <int S>
__device__ __forceinline__ void dec_stats(const uint32_t *Q, int f, int outs, int64_t cs, int64_t n_bins, double r,
                                          Run &st)
{
    const int64_t j_lo = (cs + f - 1) / f;
    int64_t j_end = (cs + outs + f - 1) / f;
    j_end = j_end < n_bins ? j_end : n_bins;
    for (int64_t jj = (int64_t)threadIdx.x * S; j_lo + jj < j_end; jj += (int64_t)blockDim.x * S) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int64_t j = j_lo + jj + s;
            if (j < j_end) {
                const int u = (int)(j * f - cs);
                run_add(st, (int32_t)(Q[u + f] - Q[u]), (uint32_t)j, r);
            }
        }
    }
}

__device__ __forceinline__ void dec_stats_any(int step, const uint32_t *Q, int f, int outs, int64_t cs,
                                              int64_t n_bins, double r, Run &st)
{
    switch (step) {
    case 1: dec_stats<1>(Q, f, outs, cs, n_bins, r, st); break;
    case 2: dec_stats<2>(Q, f, outs, cs, n_bins, r, st); break;
    case 4: dec_stats<4>(Q, f, outs, cs, n_bins, r, st); break;
    default: dec_stats<8>(Q, f, outs, cs, n_bins, r, st); break;
    }
}

__device__ __forceinline__ void width_stats_any(int step, const uint32_t *Q, int w, int outs, int64_t cs,
                                                int64_t n_valid, double r, Run &st)
{
    switch (step) {
    case 1: width_stats<1>(Q, w, outs, cs, n_valid, r, st); break;
    case 2: width_stats<2>(Q, w, outs, cs, n_valid, r, st); break;
    case 4: width_stats<4>(Q, w, outs, cs, n_valid, r, st); break;
    default: width_stats<8>(Q, w, outs, cs, n_valid, r, st); break;
    }
}

// ---- fused boxcar + S/N: one work-group per dedispersed row ----------------
// One beam per launch, or a table of beams whose rows are laid out back to
// back in the grid.
// MAXT: the work-group size bound the kernel is compiled for; smaller bounds
// leave more registers per work-item for the NW running statistics.
template <int NW, int MAXT>
__global__ __launch_bounds__(MAXT) void integrate_snr_kernel(BoxJob single, const BoxJob *__restrict__ jobs, int n_jobs,
                                                             WidthSet ws, int chunk, int halo)
{
    extern __shared__ uint4 lds4[];
    uint32_t *Q = reinterpret_cast<uint32_t *>(lds4);
    Stat *scratch = reinterpret_cast<Stat *>(lds4);  // reused after the last chunk
    __shared__ uint32_t wave_tot[16];
    int i = blockIdx.x;
    BoxJob job = single;
    if (jobs) {
        int j = 0;
        while (j + 1 < n_jobs && jobs[j + 1].row_start <= i) ++j;
        job = jobs[j];
        i -= job.row_start;
    }
    const int64_t n_out = job.n_out;
    const int32_t *__restrict__ row = job.dd + (size_t)i * job.dd_stride;
    const int outs = chunk - halo;
    const double d0 = (double)row[0];

    Run st[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) run_init(st[k]);

    for (int64_t cs = 0; cs < n_out; cs += outs) {
        load_prefix(row, cs, n_out, job.vec_ok != 0, Q, wave_tot);
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (k < ws.n) {
                const int w = ws.w[k];
                if (ws.dec)
                    dec_stats_any(ws.step[k], Q, w, outs, cs, n_out / w, d0 * w, st[k]);
                else
                    width_stats_any(ws.step[k], Q, w, outs, cs, n_out - w + 1, d0 * w, st[k]);
            }
        }
        __syncthreads();
    }
    Stat sr[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) sr[k] = run_stat(st[k]);
    block_reduce<NW>(sr, ws.n, scratch);
    if ((int)threadIdx.x < ws.n) {
        const int k = threadIdx.x;
        const int w = ws.w[k];
        finish(scratch[k * 16], ws.dec ? n_out / w : n_out - w + 1, d0 * w, job.snr + (size_t)k * job.n_dm + i,
               job.peak ? job.peak + (size_t)k * job.n_dm + i : nullptr);
    }
}

// ---- fused boxcar + S/N over wavefront spans (sliding widths) -------------
//
// One work-group per dedispersed row and W = blockDim / 64 wavefronts.  The
// row's outputs are cut into blocks of 256 (64 lanes x 4); wavefront v sweeps
// the blocks [v nb / W, (v + 1) nb / W) in order, on its own (no barrier
// until the end).  Per step j:
//  - block j + 1's samples (loaded SPAN_NB - 1 steps earlier, 16 B per lane,
//    coalesced) are centred on c = dd[row][0], prefix-summed across the
//    wavefront with DPP and written to a two-block LDS ring (slot (j + 1) & 1);
//    the first entries of slot 0 are repeated after slot 1, so that no read
//    wraps;
//  - lane l reads the prefix at its 4 outputs u = 256 j + 4 l .. + 3 and, per
//    width w, at u + w: box' = Q[u + w] - Q[u] is the width-w boxcar minus
//    w c, exact in uint32 arithmetic because its true value fits int32;
//  - per width it keeps the running maximum (3-input maxima of its 4 values),
//    the block where that maximum last rose, and the sum of squares in 64 bits
//    (one 32 x 32 + 64-bit multiply-add per value).
// A boxcar fits int32 while width x max |centred sample| does, a lane's sum of
// squares 64 bits while its square times the values per lane does, and a
// block's total int32 while max |centred sample| < 2^23; each wavefront tracks
// its largest centred sample, and a width that breaks a bound (a first sample
// far from the others, a wide boxcar and a long row together) is swept again in
// FP64 after the first sweep (span_again).  The sum of box' over the
// row needs no per-output work: it is w T minus head and tail terms, with T the
// centred row's sum.  After the sweep: wavefront reductions, one barrier, then
// per width one wavefront finds the first index of the maximum (its 4 candidate
// outputs in the earliest block that reaches it differ by the samples that
// enter and leave), forms the mean from the closed form, the variance and the
// S/N.
//
// Two forms.  Narrow (LOOK = 1): widths to 64, a window ends in the next block
// at the latest, 592 dwords of LDS per wavefront.  Wide (LOOK = 4): widths to
// 1024, 8 KiB, indices masked.  Both are bound by vector issue (about 3 per
// width and sample).  The wide form, us, with 11 widths 1 .. 1024 in place of
// two passes over LDS chunks with FP64 sums per output: 1024 rows x 24576
// samples 236 -> 60, 2048 x 12208 177 -> 65, 256 x 8192 74 -> 26; 10 uneven
// widths to 999: 297 -> 92, 219 -> 78, 89 -> 39.  10 widths to 24 take 84 as two
// narrow passes and 128 as one wide one, so the wide form is for widths above
// 64, and for more than 8 widths of a table of beams (which has no passes).

constexpr int kSpanBlk = 256;
constexpr int kSpanMaxW = 64;
constexpr int kSpanWideW = 1024;
#ifndef SPAN_NB
#define SPAN_NB 4
#endif
// reads of an odd block reach 256 + 4 * 63 + kSpanMaxW + 7 = 579 < 2 * 256 + kSpanDup
constexpr int kSpanDup = 80;
constexpr int kSpanRing = 2 * kSpanBlk + kSpanDup;  // dwords per wavefront
// The wide form (LOOK = 4): a window of up to 1024 samples ends in one of the
// four blocks after its own, so the ring holds 8 and its indices are masked.
constexpr int kSpanWideRing = 8 * kSpanBlk;

template <int LOOK>
__device__ __forceinline__ const u32x4 *span_at(const uint32_t *ring, int i)
{
    return reinterpret_cast<const u32x4 *>(ring + (LOOK == 1 ? i : i & (kSpanWideRing - 1)));
}

struct SpanRes {
    long long key;
    double s2;
};

// Inclusive prefix sum across the wavefront (rows of 16 lanes with row_shr,
// then row_bcast15 / row_bcast31 between rows).
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false); // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false); // row_bcast:31
    return v;
}

__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Raw samples of one lane in one block (block b: samples 256 b + 4 lane ..
// + 3).  VEC (16-byte aligned rows of >= 4 samples): one 16-byte load; in the
// block at the row's end a lane whose 4 samples are not all in the row re-reads
// them one by one when the block is consumed.  Otherwise four dword loads.
// Plain loads go through global-address-space pointers: flat loads would also
// count against the LDS counter, and the compiler would then drain every load in
// flight at each LDS wait.  Indices are 32-bit: the launcher takes rows of fewer
// than 2^29 samples.
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) int32_t g_i32;
typedef const __attribute__((address_space(1))) i32x4 g_i4;

// Buffer loads: a row is a buffer of n_out dwords whose reads past its end
// return zero (the hardware's range check, dword by dword: a 16-byte load that
// straddles the end returns what lies in the row), so no load needs its address
// clamped and the offsets are a fixed per-lane part plus a scalar block part.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const int32_t *row, int n_out)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(row), (short)0, n_out * 4, 0x00020000);
}

template <bool VEC>
__device__ __forceinline__ i32x4 span_load(__amdgpu_buffer_rsrc_t rs, int blk, int lane)
{
    // the whole byte offset in the vector operand, which the range check
    // covers (blk >= 0; rows of fewer than 2^29 samples)
    const int off = blk * (kSpanBlk * 4) + 16 * lane;
    if (VEC) return __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    i32x4 v;
    v.x = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
    v.y = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 4, 0, 0);
    v.z = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 8, 0, 0);
    v.w = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 12, 0, 0);
    return v;
}

__device__ __forceinline__ int32_t max3i(int32_t a, int32_t b, int32_t c)
{
    int32_t r;
    asm("v_max3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

__device__ __forceinline__ int32_t min3i(int32_t a, int32_t b, int32_t c)
{
    int32_t r;
    asm("v_min3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Centres block `blk` on c, writes its prefix (starting at `base`) to ring
// slot blk & 1, widens [xlo, xhi] to its samples and returns the
// block's total (uint32, true value fits int32).
template <bool VEC, int LOOK>
__device__ __forceinline__ uint32_t span_put(uint32_t *ring, int blk, const i32x4 &r, const int32_t *__restrict__ row,
                                             int n_out, int32_t c, uint32_t base, int lane, int32_t &xlo,
                                             int32_t &xhi)
{
    const int t = blk * kSpanBlk + 4 * lane;
    uint32_t x[4];
    auto take = [&](int32_t v0, int32_t v1, int32_t v2, int32_t v3) {
        xlo = min3i(min3i(xlo, v0, v1), v2, v3);
        xhi = max3i(max3i(xhi, v0, v1), v2, v3);
        x[0] = (uint32_t)v0 - (uint32_t)c; x[1] = (uint32_t)v1 - (uint32_t)c;
        x[2] = (uint32_t)v2 - (uint32_t)c; x[3] = (uint32_t)v3 - (uint32_t)c;
    };
    if (VEC && (blk + 1) * kSpanBlk <= n_out) {  // the whole block lies in the row
        take(r.x, r.y, r.z, r.w);
    } else if (VEC) {
        if (t + 4 <= n_out) {
            take(r.x, r.y, r.z, r.w);
        } else {
            int32_t v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (t + e < n_out) ? ((g_i32 *)row)[t + e] : c;
            take(v[0], v[1], v[2], v[3]);
        }
    } else {
        take(t < n_out ? r.x : c, t + 1 < n_out ? r.y : c, t + 2 < n_out ? r.z : c, t + 3 < n_out ? r.w : c);
    }
    const uint32_t l0 = x[0], l1 = l0 + x[1], l2 = l1 + x[2], l3 = l2 + x[3];
    const uint32_t incl = wave_scan_incl(l3);
    const uint32_t ex = incl - l3 + base;
    const u32x4 q = u32x4{ex, ex + l0, ex + l1, ex + l2};
    const int slot = blk & (LOOK == 1 ? 1 : 7);
    *reinterpret_cast<u32x4 *>(ring + slot * kSpanBlk + 4 * lane) = q;
    if (LOOK == 1 && slot == 0 && lane < kSpanDup / 4) *reinterpret_cast<u32x4 *>(ring + 2 * kSpanBlk + 4 * lane) = q;
    return (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
}

// box'[e] = Q[b + e + w] - Q[b + e] for the lane's 4 outputs: A = Q[b .. b + 3],
// g = Q[b + w - R ..], R = w & 3.
template <int R>
__device__ __forceinline__ void span_box(const uint32_t (&g)[8], const u32x4 &A, int32_t (&x)[4])
{
    x[0] = (int32_t)(g[R] - A.x); x[1] = (int32_t)(g[R + 1] - A.y);
    x[2] = (int32_t)(g[R + 2] - A.z); x[3] = (int32_t)(g[R + 3] - A.w);
}

template <bool POW2>
__device__ __forceinline__ int span_width(const WidthSet &ws, int k)
{
    return POW2 ? (1 << k) : ws.w[k];
}

// One block of one width: the lane's 4 boxcar values x, all valid (TAIL
// false) or valid below n_valid (TAIL true).  CHAIN: one multiply-add after the
// other; the compiler else adds the four products up first in some kernels, an
// addition more (widths 1 .. 1024 5 % slower; widths of any remainder, whose
// values come later, 4-10 % faster so).
template <bool TAIL, bool CHAIN>
__device__ __forceinline__ void span_acc(const int32_t (&x)[4], int t0, int n_valid, int32_t &vmax, int32_t &jmax,
                                         unsigned long long &s2, int32_t j)
{
    int32_t m;
    if (!TAIL) {
        m = max3i(max3i(vmax, x[0], x[1]), x[2], x[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s2 += (unsigned long long)((long long)x[e] * (long long)x[e]);
            if (CHAIN) asm("" : "+v"(s2));
        }
    } else {
        m = vmax;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool ok = t0 + e < n_valid;
            m = ok ? max(m, x[e]) : m;
            const int32_t v = ok ? x[e] : 0;
            s2 += (unsigned long long)((long long)v * (long long)v);
        }
    }
    jmax = m != vmax ? j : jmax;
    vmax = m;
}

// The statistics of block j for every width (its prefix and the next
// block's are in the ring).
template <int NW, bool POW2, bool TAIL, int LOOK>
__device__ __forceinline__ void span_block(const uint32_t *ring, int j, int lane, const WidthSet &ws, int n_out,
                                           int32_t (&vmax)[NW], int32_t (&jmax)[NW], unsigned long long (&s2)[NW])
{
    const int b = (j & (LOOK == 1 ? 1 : 7)) * kSpanBlk + 4 * lane;
    const int t0 = j * kSpanBlk + 4 * lane;
    if (POW2) {
        // widths 1, 2, 4, ..: every window end lies in one of the groups of
        // four at offsets 0, 4, 8, 16, ..; all of them are read before any is
        // used, so that a step waits for LDS once (read one by one, each read
        // would wait a full LDS latency)
        constexpr int NG = NW < 3 ? 2 : NW - 1;
        u32x4 G[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) G[g] = *span_at<LOOK>(ring, b + (g == 0 ? 0 : 2 << g));
        __builtin_amdgcn_sched_barrier(0);
        const u32x4 A = G[0];
        const uint32_t lo[8] = {G[0].x, G[0].y, G[0].z, G[0].w, G[1].x, G[1].y, G[1].z, G[1].w};
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            int32_t x[4];
            if (k < 2) {  // w = 1, 2: ends inside groups 0 and 1
                const int w = 1 << k;
                x[0] = (int32_t)(lo[w] - A.x); x[1] = (int32_t)(lo[w + 1] - A.y);
                x[2] = (int32_t)(lo[w + 2] - A.z); x[3] = (int32_t)(lo[w + 3] - A.w);
            } else {      // w = 4 << (k - 2): group k - 1
                const u32x4 E = G[k - 1];
                x[0] = (int32_t)(E.x - A.x); x[1] = (int32_t)(E.y - A.y);
                x[2] = (int32_t)(E.z - A.z); x[3] = (int32_t)(E.w - A.w);
            }
            span_acc<TAIL, true>(x, t0, n_out - (1 << k) + 1, vmax[k], jmax[k], s2[k], j);
        }
        return;
    }
    const u32x4 A = *reinterpret_cast<const u32x4 *>(ring + b);
    // four widths' reads at a time, all before the first use, as above (a read
    // that only one of four remainders does without costs less than a wait)
#pragma unroll
    for (int k0 = 0; k0 < NW; k0 += 4) {
        if (LOOK > 1 && k0 >= ws.n) continue;  // (the wide form is compiled for several counts at once)
        u32x4 lo[4], hi[4];
#pragma unroll
        for (int q = 0; q < 4 && k0 + q < NW; ++q) {
            const int at = b + (span_width<POW2>(ws, k0 + q) & ~3);
            lo[q] = *span_at<LOOK>(ring, at);
            hi[q] = *span_at<LOOK>(ring, at + 4);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4 && k0 + q < NW; ++q) {
            const int k = k0 + q;
            if (LOOK > 1 && k >= ws.n) continue;
            const int w = span_width<POW2>(ws, k);
            const uint32_t g[8] = {lo[q].x, lo[q].y, lo[q].z, lo[q].w, hi[q].x, hi[q].y, hi[q].z, hi[q].w};
            int32_t x[4];
            switch (w & 3) {
            case 0: span_box<0>(g, A, x); break;
            case 1: span_box<1>(g, A, x); break;
            case 2: span_box<2>(g, A, x); break;
            default: span_box<3>(g, A, x); break;
            }
            span_acc<TAIL, false>(x, t0, n_out - w + 1, vmax[k], jmax[k], s2[k], j);
        }
    }
}

// Whole-wavefront reductions with DPP (quad permutes, row mirrors, then
// row_bcast15 / row_bcast31 into the last row); the result is read from lane
// 63 and is the same in every lane.  64-bit values move as two halves.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp64(uint64_t v, uint64_t identity)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)identity, (int)(uint32_t)v, CTRL, ROWS,
                                                               0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(identity >> 32), (int)(uint32_t)(v >> 32),
                                                               CTRL, ROWS, 0xf, false);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t lane63(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ long long wave_max_ll(long long v)
{
    const uint64_t id = (uint64_t)LLONG_MIN;
    auto mx = [](long long a, uint64_t b) { return a > (long long)b ? a : (long long)b; };
    v = mx(v, dpp64<0xb1, 0xf>((uint64_t)v, id));   // quad_perm [1,0,3,2]
    v = mx(v, dpp64<0x4e, 0xf>((uint64_t)v, id));   // quad_perm [2,3,0,1]
    v = mx(v, dpp64<0x141, 0xf>((uint64_t)v, id));  // row_half_mirror
    v = mx(v, dpp64<0x140, 0xf>((uint64_t)v, id));  // row_mirror
    v = mx(v, dpp64<0x142, 0xa>((uint64_t)v, id));  // row_bcast:15
    v = mx(v, dpp64<0x143, 0xc>((uint64_t)v, id));  // row_bcast:31
    return (long long)lane63((uint64_t)v);
}

__device__ __forceinline__ double wave_sum_d(double v)
{
    auto add = [](double a, uint64_t b) { return a + __longlong_as_double((long long)b); };
    auto bits = [](double a) { return (uint64_t)__double_as_longlong(a); };
    v = add(v, dpp64<0xb1, 0xf>(bits(v), 0));
    v = add(v, dpp64<0x4e, 0xf>(bits(v), 0));
    v = add(v, dpp64<0x141, 0xf>(bits(v), 0));
    v = add(v, dpp64<0x140, 0xf>(bits(v), 0));
    v = add(v, dpp64<0x142, 0xa>(bits(v), 0));
    v = add(v, dpp64<0x143, 0xc>(bits(v), 0));
    return __longlong_as_double((long long)lane63(bits(v)));
}

// f(K) for K = 0 .. N - 1 as constants (a loop of this size is not always
// unrolled, and the statistics it indexes would then live in memory).
template <typename F, int... K>
__device__ __forceinline__ void each_of(F f, std::integer_sequence<int, K...>)
{
    (f(std::integral_constant<int, K>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(F f)
{
    each_of(f, std::make_integer_sequence<int, N>{});
}

// Statistics in the form that reductions move between lanes: the maximum, ~(its
// first sample), and sums.
struct DecStat {
    int32_t v;
    uint32_t nt;
    double s1, s2;
};
struct SpanStat {
    int32_t v;
    uint32_t nt;
    double s2;
};

template <typename S>
__device__ __forceinline__ long long lane_key(const S &a)
{
    return (long long)(((uint64_t)(uint32_t)a.v << 32) | a.nt);
}

template <typename S>
__device__ __forceinline__ void merge_max(S &a, const S &b)
{
    const bool up = lane_key(b) > lane_key(a);
    a.v = up ? b.v : a.v;
    a.nt = up ? b.nt : a.nt;
}
__device__ __forceinline__ void merge(DecStat &a, const DecStat &b)
{
    merge_max(a, b);
    a.s1 += b.s1;
    a.s2 += b.s2;
}
__device__ __forceinline__ void merge(SpanStat &a, const SpanStat &b)
{
    merge_max(a, b);
    a.s2 += b.s2;
}

// f(x, y) on the dwords of two statistics.
template <typename S, typename F>
__device__ __forceinline__ void dwords(S &a, S &b, F f)
{
    struct D {
        uint32_t w[sizeof(S) / 4];
    };
    D x = __builtin_bit_cast(D, a), y = __builtin_bit_cast(D, b);
#pragma unroll
    for (unsigned i = 0; i < sizeof(S) / 4; ++i) f(x.w[i], y.w[i]);
    a = __builtin_bit_cast(S, x);
    b = __builtin_bit_cast(S, y);
}

// One step of the reduction within rows of 16 lanes.
template <int CTRL, typename S>
__device__ __forceinline__ void row_step(S &a)
{
    S b = a;
    dwords(a, b, [](uint32_t &, uint32_t &y) {
        y = (uint32_t)__builtin_amdgcn_update_dpp((int)y, (int)y, CTRL, 0xf, 0xf, false);
    });
    merge(a, b);
}

// Reduces N (a multiple of 4) statistics over the wavefront; out(k, total) runs
// in one lane for each k.  Two steps halve the number of statistics each, by
// exchanging halves of two of them at a time; then each row of 16 lanes holds
// one of four, 4 a + 2 (row & 1) + (row >> 1).  (One by one, ten statistics took
// twice the sweep of a row of 12208 samples.)
template <int N, typename S, typename F>
__device__ __forceinline__ void wave_reduce_all(S (&d)[N], int lane, F out)
{
    each<N / 2>([&](auto M) {
        dwords(d[2 * M], d[2 * M + 1], [](uint32_t &x, uint32_t &y) {
            const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
            x = r[0];
            y = r[1];
        });
        merge(d[2 * M], d[2 * M + 1]);
    });
    each<N / 4>([&](auto A) {
        S &t = d[4 * A];
        dwords(t, d[4 * A + 2], [](uint32_t &x, uint32_t &y) {
            const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
            x = r[0];
            y = r[1];
        });
        merge(t, d[4 * A + 2]);
        row_step<0xb1>(t);   // quad_perm [1,0,3,2]
        row_step<0x4e>(t);   // quad_perm [2,3,0,1]
        row_step<0x141>(t);  // row_half_mirror
        row_step<0x140>(t);  // row_mirror
        const int r = lane >> 4;
        if ((lane & 15) == 0) out(4 * A + 2 * (r & 1) + (r >> 1), t);
    });
}

// The statistics of the widths in `again` (bits) over a wavefront's blocks
// [jb, je) once more, of the samples as they are (where a boxcar of them fits
// int32) and in FP64 about the boxcar of c: up to 4 widths per sweep.  Leaves in
// res the maximum with its first index and the sum of squares, in s1 the sum.
// 1024 rows x 200000 samples that begin with 0, us: widths 1 .. 1024 2720 ->
// 590, width 1024 alone 2940 -> 360 (before, one wavefront slid each such window
// along its row, uncoalesced; LDS chunks in FP64 take 1900 and 490).
template <int NW, bool POW2, bool VEC, int LOOK>
__device__ __forceinline__ void span_again(uint32_t again, uint32_t *ring, const int32_t *__restrict__ row,
                                           __amdgpu_buffer_rsrc_t rs, int n_out, int32_t c, int jb, int je, int lane,
                                           const WidthSet &ws, SpanRes *res, double *s1)
{
    constexpr int kTogether = 2;
    while (again) {
        int width[kTogether], at[kTogether], n = 0;
        Run st[kTogether];
#pragma unroll
        for (int q = 0; q < kTogether; ++q) {
            run_init(st[q]);
            width[q] = at[q] = 0;
            if (!again) continue;
            at[q] = __builtin_ctz(again);
            width[q] = POW2 ? 1 << at[q] : ws.w[at[q]];
            again &= again - 1;
            ++n;
        }
        uint32_t base = 0;
        int32_t lo = 0, hi = 0;
        auto put = [&](int blk) {
            base += span_put<VEC, LOOK>(ring, blk, span_load<VEC>(rs, blk, lane), row, n_out, 0, base, lane, lo, hi);
        };
        if (jb < je)
            for (int m = 0; m < LOOK; ++m) put(jb + m);
#pragma unroll 1
        for (int j = jb; j < je; ++j) {
            put(j + LOOK);
            wave_sync_lds();
            const int b = (j & (LOOK == 1 ? 1 : 7)) * kSpanBlk + 4 * lane, t0 = j * kSpanBlk + 4 * lane;
#pragma unroll
            for (int q = 0; q < kTogether; ++q) {
                if (q >= n) continue;
                const double r = (double)c * (double)width[q];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int to = b + e + width[q];
                    const uint32_t x = ring[LOOK == 1 ? to : to & (kSpanWideRing - 1)] - ring[b + e];
                    if (t0 + e <= n_out - width[q]) run_add(st[q], (int32_t)x, (uint32_t)(t0 + e), r);
                }
            }
            wave_sync_lds();
        }
#pragma unroll
        for (int q = 0; q < kTogether; ++q) {
            if (q >= n) continue;
            const Stat t = wave_reduce(run_stat(st[q]));
            if (lane == 0) {
                res[at[q]] = SpanRes{t.key, t.s2};
                s1[at[q]] = t.s1;
            }
        }
    }
}

// NW: the number of widths (LOOK = 4 without POW2: at least); POW2: widths are
// 1, 2, 4, ... 2^(NW-1).  LOOK: blocks after its own that a window may end in.
constexpr int NB = SPAN_NB;
template <int NW, bool POW2, bool VEC, int LOOK>
__global__ __launch_bounds__(LOOK == 1 ? 1024 : 512) __attribute__((amdgpu_waves_per_eu(LOOK == 1 || NW == 11 ? 4 : 2)))
void span_snr_kernel(BoxJob single, const BoxJob *__restrict__ jobs, int n_jobs, WidthSet ws)
{
    extern __shared__ uint4 lds4[];
    // the wavefront index is uniform: keep it (and the span bounds, the block
    // counter and every branch on them) in scalar registers
    const int W = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    constexpr int kRing = LOOK == 1 ? kSpanRing : kSpanWideRing;
    uint32_t *ring = reinterpret_cast<uint32_t *>(lds4) + wave * kRing;
    SpanRes *res = reinterpret_cast<SpanRes *>(reinterpret_cast<uint32_t *>(lds4) + W * kRing);
    long long *tres = reinterpret_cast<long long *>(res + W * NW);
    long long *peaks = tres + W;  // per wavefront: its largest centred sample
    double *sums = reinterpret_cast<double *>(peaks + W);  // per wavefront and width, of those swept again

    int i = blockIdx.x;
    BoxJob job = single;
    if (jobs) {
        int j = 0;
        while (j + 1 < n_jobs && jobs[j + 1].row_start <= i) ++j;
        job = jobs[j];
        i -= job.row_start;
    }
    const int n_out = (int)job.n_out;
    const int32_t *__restrict__ row = job.dd + (size_t)i * job.dd_stride;
    const int32_t c = *(g_i32 *)row;
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(row, n_out);
    // the row's first and last 64 samples (for the boxcar sums' head and tail
    // terms), loaded now and used after the sweep
    const int32_t head = lane < n_out ? ((g_i32 *)row)[lane] : 0;
    const int32_t tail = n_out - 1 - lane >= 0 ? ((g_i32 *)row)[n_out - 1 - lane] : 0;
    int maxw = 1;
#pragma unroll
    for (int k = 0; k < NW; ++k)
        if (LOOK == 1 || k < ws.n) maxw = max(maxw, span_width<POW2>(ws, k));
    const int n_min = n_out - maxw + 1;  // outputs below it are valid for every width

    int32_t vmax[NW], jmax[NW];
    unsigned long long s2[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        vmax[k] = INT32_MIN;
        jmax[k] = -1;
        s2[k] = 0;
    }
    long long tsum = 0;
    int32_t xlo = c, xhi = c;

    const int nb = (n_out + kSpanBlk - 1) / kSpanBlk;
    const int jb = (int)((uint32_t)nb * (uint32_t)wave / (uint32_t)W),
              je = (int)((uint32_t)nb * (uint32_t)(wave + 1) / (uint32_t)W);
    if (jb < je) {
        // blocks before j_tail have every output valid for every width; the
        // others (at most LOOK + 1, at the row's end) take the masked statistics
        const int j_tail = min(max(n_min / kSpanBlk, jb), je);
        uint32_t base = 0;
        auto put = [&](int blk, const i32x4 &x) {
            const uint32_t tot = span_put<VEC, LOOK>(ring, blk, x, row, n_out, c, base, lane, xlo, xhi);
            base += tot;
            if (blk >= jb && blk < je) tsum += (int32_t)tot;
        };
        // the first LOOK blocks from j on, loaded together
        auto begin = [&](int j) {
            i32x4 first[LOOK];
#pragma unroll
            for (int m = 0; m < LOOK; ++m) first[m] = span_load<VEC>(rs, max(j + m, 0), lane);
#pragma unroll
            for (int m = 0; m < LOOK; ++m) put(j + m, first[m]);
        };
        // Main part, blocks [jb, j_tail): NB block buffers.  While block j
        // is summed, blocks to j + LOOK (its windows' lookahead, put into the
        // ring first) are there and the NB - 1 after it are being loaded.  The
        // loop is unrolled NB times so that buffers are never copied (a copy
        // would wait for the load in flight); it starts NB - 1 steps early at
        // most (dummy steps: loads and prefix writes of earlier blocks, no
        // statistics), so that its length is a multiple of NB.
        if (jb < j_tail) {
            const int r = (NB - (j_tail - jb) % NB) % NB;
            int j = jb - r;
            i32x4 buf[NB];
#pragma unroll
            for (int u = 1; u < NB; ++u) buf[u] = span_load<VEC>(rs, max(j + LOOK - 1 + u, 0), lane);
            begin(j);
            for (; j < j_tail; j += NB) {
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int jj = j + u;
                    // blocks past the lookahead are loaded and never used
                    // (past the row's end the loads return zeros)
                    buf[u] = span_load<VEC>(rs, max(jj + LOOK - 1 + NB, 0), lane);
                    put(jj + LOOK, buf[(u + 1) % NB]);
                    wave_sync_lds();
                    if (jj >= jb) span_block<NW, POW2, false, LOOK>(ring, jj, lane, ws, n_out, vmax, jmax, s2);
                    wave_sync_lds();
                }
            }
        } else {
            begin(jb);
        }
        // tail blocks: the last lookahead block loaded and put, then block
        // j's masked statistics
        for (int j = j_tail; j < je; ++j) {
            put(j + LOOK, span_load<VEC>(rs, j + LOOK, lane));
            wave_sync_lds();
            span_block<NW, POW2, true, LOOK>(ring, j, lane, ws, n_out, vmax, jmax, s2);
            wave_sync_lds();
        }
    }
    // the largest centred sample (of this wavefront's)
    uint32_t far = max((uint32_t)xhi - (uint32_t)c, (uint32_t)c - (uint32_t)xlo);
    far = max(far, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)far, 0xb1, 0xf, 0xf, false));
    far = max(far, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)far, 0x4e, 0xf, 0xf, false));
    far = max(far, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)far, 0x141, 0xf, 0xf, false));
    far = max(far, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)far, 0x140, 0xf, 0xf, false));
    far = max(max((uint32_t)__builtin_amdgcn_readlane((int)far, 0), (uint32_t)__builtin_amdgcn_readlane((int)far, 16)),
              max((uint32_t)__builtin_amdgcn_readlane((int)far, 32), (uint32_t)__builtin_amdgcn_readlane((int)far, 48)));
    long long xmax = far;

    // wavefront totals: per width (max, earliest 4-output group) and sum of squares
    constexpr int NP = (NW + 3) / 4 * 4;
    SpanStat d[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        if (k < NW)
            d[k] = SpanStat{vmax[k], ~(uint32_t)(jmax[k] >= 0 ? jmax[k] * kSpanBlk + 4 * lane : 0),
                            (double)s2[k]};
        else
            d[k] = SpanStat{INT32_MIN, 0u, 0.0};
    }
    wave_reduce_all(d, lane, [&](int k, const SpanStat &t) {
        if (k < NW) res[wave * NW + k] = SpanRes{lane_key(t), t.s2};
    });
    if (lane == 0) {
        tres[wave] = tsum;
        peaks[wave] = xmax;
    }
    __syncthreads();
    long long T = 0;
    for (int v = 0; v < W; ++v) {
        xmax = max(xmax, peaks[v]);
        T += tres[v];
    }
    const int blocks = (nb + W - 1) / W;
    // Exact: a block's total (256 centred samples) and a boxcar fit int32, and a
    // lane's sum of squares (at most 4 values a block) 64 bits.
    auto exact = [&](int w) {
        const double bound = (double)w * (double)xmax;
        return xmax < (1 << 23) && bound < 2147483647.0 && bound * bound * (4.0 * (double)blocks) < 1.8e19;
    };
    uint32_t again = 0, slow = 0;  // widths to sweep again, and those that no sweep holds
    if (__builtin_expect(!exact(maxw), 0)) {
#pragma unroll 1
        for (int k = 0; k < (LOOK == 1 ? NW : ws.n); ++k) {
            const int w = span_width<POW2>(ws, k);
            if (exact(w)) continue;
            // (where boxcars of the samples themselves fit int32)
            if ((double)w * ((double)xmax + fabs((double)c)) < 2147483648.0)
                again |= 1u << k;
            else
                slow |= 1u << k;
        }
        again = (uint32_t)__builtin_amdgcn_readfirstlane((int)again);
        slow = (uint32_t)__builtin_amdgcn_readfirstlane((int)slow);
        span_again<NW, POW2, VEC, LOOK>(again, ring, row, rs, n_out, c, jb, je, lane, ws, res + wave * NW,
                                        sums + wave * NW);
        __syncthreads();
    }
    // this wavefront's widths k = wave, wave + W, ..: totals over the
    // wavefronts (in a fixed order), then the loads that find the first index
    // of each maximum among outputs u0 .. u0 + 3 (the samples that enter and
    // leave from one to the next), all issued before any is used
    long long key[NW];
    double s2t[NW];
    int32_t edge[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        if (k % W != wave || (LOOK > 1 && k >= ws.n)) continue;
        key[k] = LLONG_MIN;
        s2t[k] = 0.0;
        for (int v = 0; v < W; ++v) {
            const SpanRes r = res[v * NW + k];
            key[k] = r.key > key[k] ? r.key : key[k];
            s2t[k] += r.s2;
        }
        const int u0 = (int)(0xffffffffu - (uint32_t)(key[k] & 0xffffffffll));
        const int at = u0 + (lane < 3 ? lane : span_width<POW2>(ws, k) + lane - 3);
        edge[k] = (lane < 6 && at < n_out) ? row[at] : 0;
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        if (k % W != wave || (LOOK > 1 && k >= ws.n)) continue;
        const int w = span_width<POW2>(ws, k);
        const int N = n_out - w + 1;
        double vm = (double)(int32_t)(key[k] >> 32);
        int tstar = (int)(0xffffffffu - (uint32_t)(key[k] & 0xffffffffll));
        double s1, s = s2t[k];
        if ((again >> k) & 1u) {
            s1 = 0.0;
            for (int v = 0; v < W; ++v) s1 += sums[v * NW + k];
            vm -= (double)w * (double)c;
        } else if (!((slow >> k) & 1u)) {
            // the boxcar sum's weights below w: its head's and tail's samples
            double corr = 0.0;
            auto ends = [&](int m, int32_t xh, int32_t xt) {
                const int th = m, tt = n_out - 1 - m;
                if (th < n_out) {
                    const int cnt = min(th, N - 1) - max(0, th - w + 1) + 1;
                    corr += (double)(w - cnt) * (double)(xh - c);
                }
                if (tt >= w - 1) {
                    const int cnt = min(tt, N - 1) - max(0, tt - w + 1) + 1;
                    corr += (double)(w - cnt) * (double)(xt - c);
                }
            };
            if (lane <= w - 2) ends(lane, head, tail);
            if (LOOK > 1) {
                // (w <= n_out: both indices lie in the row)
                for (int m = 64 + lane; m <= w - 2; m += 64) ends(m, row[m], row[n_out - 1 - m]);
            }
            corr = wave_sum_d(corr);
            s1 = (double)w * (double)T - corr;
            // box[u0 + e] - box[u0], and the first e of the largest
            long long d = 0, best = 0;
            const int u0 = tstar;
#pragma unroll
            for (int e = 1; e < 4; ++e) {
                d += (long long)__builtin_amdgcn_readlane(edge[k], e + 2) - __builtin_amdgcn_readlane(edge[k], e - 1);
                if (u0 + e < N && d > best) {
                    best = d;
                    tstar = u0 + e;
                }
            }
        } else {
            // any samples: lane l takes a contiguous run of outputs and slides
            // its window along it, in int64 and FP64
            const int C = (N + 63) / 64, t0 = lane * C, t1 = min(N, t0 + C);
            long long top = LLONG_MIN;
            int at = 0x7fffffff;
            double a1 = 0.0, a2 = 0.0;
            if (t0 < t1) {
                long long bx = 0;
                for (int m = 0; m < w; ++m) bx += (long long)row[t0 + m] - c;
                for (int t = t0;;) {
                    if (bx > top) {
                        top = bx;
                        at = t;
                    }
                    a1 += (double)bx;
                    a2 += (double)bx * (double)bx;
                    if (++t >= t1) break;
                    bx += (long long)row[t + w - 1] - (long long)row[t - 1];
                }
            }
            const long long most = wave_max_ll(top);
            tstar = -(int)wave_max_ll(top == most ? -(long long)at : LLONG_MIN);
            s1 = wave_sum_d(a1);
            s = wave_sum_d(a2);
            vm = (double)most;
        }
        if (lane == 0) {
            const double m1 = s1 / (double)N;
            double var = s / (double)N - m1 * m1;
            var = var > 0.0 ? var : 0.0;
            const double sigma = sqrt(var);
            job.snr[(size_t)k * job.n_dm + i] = sigma > 0.0 ? (float)((vm - m1) / sigma) : 0.0f;
            if (job.peak) job.peak[(size_t)k * job.n_dm + i] = tstar;
        }
    }
}

// ---- decimated series and their S/N over wavefront spans --------------------
//
// One work-group per dedispersed row; its wavefronts take consecutive spans of
// whole chunks of 1024 samples and sweep them without a barrier.  Per chunk: 4
// blocks of 256 samples (loaded one chunk ahead, 16 B per lane) are prefix-
// summed across the wavefront and written to LDS, the prefix running on over
// the span (uint32, modulo 2^32).  A bin of factor f is the difference of the
// prefix at two neighbouring multiples of f; the one before the chunk's first
// was kept in LDS.  Factor 1 (every sample a bin) takes its values from the
// loaded registers.  A span's samples before its first multiple of f and from
// its last one on are parts of bins that cross spans: they are put together at
// the end, where the work-group's statistics are.  So no sample is read twice
// and any factor needs the same LDS.
//
// 2048 x 12208 samples, ladder 1, 10, 20, .. 3200: 213 -> 40 us (before: two
// passes over chunks overlapping by the largest factor, three barriers each).
// The 100 MB alone take 20 us, which factors 1 or 10 by themselves meet; each
// further factor adds 2 us of vector issue and LDS latency, in iterations that
// have few bins and in the reduction.
constexpr int kDecBlocks = 4;
constexpr int kDecChunk = kDecBlocks * kSpanBlk;

// What a wavefront leaves of one factor.
struct DecRes {
    Stat st;        // its peak in samples
    uint32_t head;  // the samples before its first boundary
    uint32_t pad;
};

template <bool VEC>
__device__ __forceinline__ void dec_load(__amdgpu_buffer_rsrc_t rs, int s0, int n_out, int lane,
                                         i32x4 (&x)[kDecBlocks])
{
#pragma unroll
    for (int q = 0; q < kDecBlocks; ++q) {
        const int blk = s0 / kSpanBlk + q;
        // (16-byte loads over the row's end too would return the same, and
        // measured 1 % slower: 2048 rows x 12208 samples 41.3 us against 40.9)
        if (VEC && (blk + 1) * kSpanBlk <= n_out)
            x[q] = span_load<true>(rs, blk, lane);
        else
            x[q] = span_load<false>(rs, blk, lane);
    }
}

// NW: at least the number of factors, a multiple of 4.  A factor 1 comes first;
// step[k] is factor k's place in the results.
template <int NW, bool VEC>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NW <= 12 ? 4 : 2))) void dec_snr_kernel(BoxJob job, WidthSet ws)
{
    extern __shared__ uint4 lds4[];
    const int W = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint32_t *P = reinterpret_cast<uint32_t *>(lds4) + wave * (kDecChunk + AMBER_MAX_WIDTHS);
    uint32_t *last = P + kDecChunk;  // per factor: the prefix at the last boundary passed
    DecRes *res = reinterpret_cast<DecRes *>(reinterpret_cast<uint32_t *>(lds4) + W * (kDecChunk + AMBER_MAX_WIDTHS));
    uint32_t *total = reinterpret_cast<uint32_t *>(res + W * NW);  // the spans' sums
    const int i = blockIdx.x, n_out = (int)job.n_out;
    const int32_t *__restrict__ row = job.dd + (size_t)i * job.dd_stride;
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(row, n_out);
    const double c = (double)*(g_i32 *)row;
    const int chunks = (n_out + kDecChunk - 1) / kDecChunk;
    const int s_begin = (int)((int64_t)chunks * wave / W) * kDecChunk,
              s_end = (int)((int64_t)chunks * (wave + 1) / W) * kDecChunk;

    Run st[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) run_init(st[k]);
    const bool one = ws.w[0] == 1;
    int at[NW];  // each factor's next boundary
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const int f = k < ws.n ? ws.w[k] : 1;
        at[k] = (s_begin + f - 1) / f * f;
    }
    if (lane < NW) last[lane] = 0;
    uint32_t base = 0;
    i32x4 x[kDecBlocks];
    if (s_begin < s_end) dec_load<VEC>(rs, s_begin, n_out, lane, x);
    for (int s0 = s_begin; s0 < s_end; s0 += kDecChunk) {
        wave_sync_lds();
#pragma unroll
        for (int q = 0; q < kDecBlocks; ++q) {
            const uint32_t l0 = (uint32_t)x[q].x, l1 = l0 + (uint32_t)x[q].y, l2 = l1 + (uint32_t)x[q].z,
                           l3 = l2 + (uint32_t)x[q].w;
            const uint32_t incl = wave_scan_incl(l3);
            const uint32_t ex = incl - l3 + base;
            *reinterpret_cast<u32x4 *>(P + q * kSpanBlk + 4 * lane) = u32x4{ex, ex + l0, ex + l1, ex + l2};
            base += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        if (one) {
#pragma unroll
            for (int q = 0; q < kDecBlocks; ++q) {
                const int t = s0 + q * kSpanBlk + 4 * lane;
                const int32_t v[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
                if (s0 + (q + 1) * kSpanBlk <= n_out) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) run_add(st[0], v[e], (uint32_t)(t + e), c);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (t + e < n_out) run_add(st[0], v[e], (uint32_t)(t + e), c);
                }
            }
        }
        // (the registers are free: the next chunk's loads; past the span they
        // are never used, past the row they return zeros)
        dec_load<VEC>(rs, s0 + kDecChunk, n_out, lane, x);
        wave_sync_lds();
        each<NW>([&](auto K) {
            constexpr int k = K;
            if (k >= ws.n || (k == 0 && one)) return;
            const int f = ws.w[k];
            while (at[k] < s0 + kDecChunk && at[k] <= n_out) {
                // boundaries at[k] + lane f of this chunk; the bin that ends there
                const int b = at[k] + lane * f;
                const bool in = b < s0 + kDecChunk && b <= n_out;
                const uint32_t end = in ? P[b - s0] : 0u;
                const uint32_t from = !in || b - f < s0 ? last[k] : P[b - f - s0];
                const int n = (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(in));
                // (the span's first boundary ends another span's bin, or none)
                if (in && b - f >= s_begin) run_add(st[k], (int32_t)(end - from), (uint32_t)(b - f), c * f);
                if (lane == n - 1) last[k] = end;
                if (b < s_begin + f && in) res[wave * NW + k].head = end;
                at[k] += n * f;
                wave_sync_lds();
            }
        });
    }
    DecStat d[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) d[k] = DecStat{st[k].vmax, ~st[k].tmax, st[k].s1, st[k].s2};
    wave_reduce_all(d, lane, [&](int k, const DecStat &t) { res[wave * NW + k].st = Stat{lane_key(t), t.s1, t.s2}; });
    if (lane == 0) total[wave] = base;
    __syncthreads();
    const int k = threadIdx.x;
    if (k < ws.n) {
        const int f = ws.w[k];
        const double r = c * f;
        Stat tot;
        stat_init(tot);
        uint32_t open = 0;  // the samples so far of the bin that crosses into the next span
        for (int v = 0; v < W; ++v) {
            const DecRes &q = res[v * NW + k];
            tot.key = q.st.key > tot.key ? q.st.key : tot.key;
            tot.s1 += q.st.s1;
            tot.s2 += q.st.s2;
            if (k == 0 && one) continue;
            const int vb = (int)((int64_t)chunks * v / W) * kDecChunk, ve = (int)((int64_t)chunks * (v + 1) / W) * kDecChunk;
            const int b = (vb + f - 1) / f * f;  // the span's first boundary
            if (b < ve && b <= n_out) {
                open += q.head;
                if (b > 0) stat_add(tot, (int32_t)open, b - f, r);
                open = total[v] - (reinterpret_cast<uint32_t *>(lds4) + v * (kDecChunk + AMBER_MAX_WIDTHS) + kDecChunk)[k];
            } else {
                open += total[v];
            }
        }
        // the last boundary is the end of the last chunk: no span has it
        if (!(k == 0 && one) && n_out % kDecChunk == 0 && n_out % f == 0) stat_add(tot, (int32_t)open, n_out - f, r);
        // (peaks so far in samples)
        const uint32_t t = 0xffffffffu - (uint32_t)(tot.key & 0xffffffffll);
        tot.key = pack_key((int32_t)(tot.key >> 32), t / (uint32_t)f);
        const size_t out = (size_t)ws.step[k] * job.n_dm + i;
        finish(tot, n_out / f, r, job.snr + out, job.peak ? job.peak + out : nullptr);
    }
}

// ---- materialised boxcar: one work-group per (chunk, row) ------------------
__global__ __launch_bounds__(1024) void integrate_kernel(const int32_t *__restrict__ dd, int n_dm, int64_t dd_stride,
                                                         int64_t n_out, WidthSet ws, int chunk, int halo, int vec_ok,
                                                         int32_t *__restrict__ box, int64_t box_stride)
{
    extern __shared__ uint4 lds4[];
    uint32_t *Q = reinterpret_cast<uint32_t *>(lds4);
    __shared__ uint32_t wave_tot[16];
    const int i = blockIdx.y;
    const int outs = chunk - halo;
    const int64_t cs = (int64_t)blockIdx.x * outs;
    load_prefix(dd + (size_t)i * dd_stride, cs, n_out, vec_ok != 0, Q, wave_tot);
    for (int k = 0; k < ws.n; ++k) {
        const int w = ws.w[k];
        int32_t *__restrict__ out = box + ((size_t)k * n_dm + i) * box_stride;
        if (ws.dec) {
            // bins j whose first sample j w lies in this chunk's outputs
            const int64_t j_lo = (cs + w - 1) / w, n_bins = n_out / w;
            int64_t j_end = (cs + outs + w - 1) / w;
            j_end = j_end < n_bins ? j_end : n_bins;
            for (int64_t j = j_lo + threadIdx.x; j < j_end; j += blockDim.x) {
                const int u = (int)(j * w - cs);
                out[j] = (int32_t)(Q[u + w] - Q[u]);
            }
        } else {
            const int64_t n_valid = n_out - w + 1;
            for (int u = threadIdx.x; u < outs; u += blockDim.x) {
                const int64_t t = cs + u;
                if (t < n_valid) out[t] = (int32_t)(Q[u + w] - Q[u]);
            }
        }
    }
}

// ---- S/N of materialised boxcar series: one work-group per (row, width) ----
//
// Wavefront v takes blocks v, v + W, .. of 256 values (16 B per lane), four at a
// time, all loads before the first use.  Per value: a 3-input maximum for two,
// and FP64 sums about the row's first value; per block the group of four where
// the maximum last rose, whose first index is found at the end.  Bound by
// reading: 512 rows x 7 widths x 12208 values (175 MB) 78 -> 35 us; before, 8
// consecutive dwords per work-item with a 64-bit maximum key per value.
template <bool VEC>
__global__ __launch_bounds__(1024) void snr_kernel(const int32_t *__restrict__ box, int n_dm, int64_t box_stride,
                                                   int64_t n_out, WidthSet ws, float *__restrict__ snr,
                                                   int32_t *__restrict__ peak)
{
    __shared__ Stat scratch[16];
    const int i = blockIdx.x, k = blockIdx.y;
    const int64_t n = n_out - ws.w[k] + 1, whole = n / kSpanBlk;
    const int32_t *__restrict__ row = box + ((size_t)k * n_dm + i) * box_stride;
    const double r = (double)row[0];
    const int W = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    Run st;  // tmax: the first of the four values
    run_init(st);
    auto add = [&](const int32_t (&x)[4], int64_t t) {
        const int32_t m = max3i(max3i(st.vmax, x[0], x[1]), x[2], x[3]);
        st.tmax = m != st.vmax ? (uint32_t)t : st.tmax;
        st.vmax = m;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double d = (double)x[e] - r;
            st.s1 += d;
            st.s2 = fma(d, d, st.s2);
        }
    };
    constexpr int kAhead = 4;
    for (int64_t b = wave; b < whole; b += (int64_t)kAhead * W) {
        int32_t x[kAhead][4];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            // (past the last whole block: that one again, not used)
            const int64_t at = b + (int64_t)u * W < whole ? b + (int64_t)u * W : b;
            const g_i32 *p = (g_i32 *)row + at * kSpanBlk + 4 * lane;
            if (VEC) {
                const i32x4 v = *(const g_i4 *)p;
                x[u][0] = v.x; x[u][1] = v.y; x[u][2] = v.z; x[u][3] = v.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) x[u][e] = p[e];
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (b + (int64_t)u * W < whole) add(x[u], (b + (int64_t)u * W) * kSpanBlk + 4 * lane);
    }
    if (wave == whole % W) {
        // the rest of the row, fewer than 256 values
        for (int e = 0; e < 4; ++e) {
            const int64_t t = whole * kSpanBlk + 4 * lane + e;
            if (t >= n) break;
            const int32_t v = row[t];
            if (v > st.vmax) {
                st.vmax = v;
                st.tmax = (uint32_t)(t - e);
            }
            const double d = (double)v - r;
            st.s1 += d;
            st.s2 = fma(d, d, st.s2);
        }
    }
    Stat arr[1] = {run_stat(st)};
    block_reduce<1>(arr, 1, scratch);
    if (threadIdx.x == 0) {
        Stat s = scratch[0];
        const int32_t vmax = (int32_t)(s.key >> 32);
        // a row of INT32_MIN alone: no value rose above the maximum's start, so
        // no group was noted, and the first is the one
        const uint32_t t0 = s.key == LLONG_MIN ? 0u : 0xffffffffu - (uint32_t)(s.key & 0xffffffffll);
        // (the three loads together)
        const int64_t end = n - 1;
        const int32_t v0 = row[t0], v1 = row[(int64_t)t0 + 1 < end ? (int64_t)t0 + 1 : end],
                      v2 = row[(int64_t)t0 + 2 < end ? (int64_t)t0 + 2 : end];
        s.key = pack_key(vmax, t0 + (v0 == vmax ? 0 : v1 == vmax ? 1 : v2 == vmax ? 2 : 3));
        finish(s, n, r, snr + (size_t)k * n_dm + i, peak ? peak + (size_t)k * n_dm + i : nullptr);
    }
}

WidthSet make_widths(const amber_tiles &t, const int32_t *widths, int n, int decimate)
{
    WidthSet ws{};
    ws.dec = decimate ? 1 : 0;
    for (int k = 0; k < n; ++k) {
        ws.w[k] = widths[k];
        ws.step[k] = t.boxcar_step[k];
    }
    ws.n = n;
    return ws;
}

int halo_of(const BoxcarPlan &p) { return (p.maxw + 15) / 16 * 16; }

amber_status check_chunk(const BoxcarPlan &p)
{
    // plan_boxcar guarantees chunk >= 2 * halo; keep the launchers safe on their own
    if (p.chunk < 2 * halo_of(p)) return fail(AMBER_E_CONFIG, "boxcar chunk shorter than twice its halo");
    return AMBER_OK;
}

template <typename F>
amber_status allow_lds(F fn, int64_t bytes, const char *what)
{
    if (bytes > 64 * 1024)
        AMBER_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)bytes),
                  what);
    return AMBER_OK;
}

}  // namespace

BoxJob make_box_job(const int32_t *d_dd, int n_dm, int64_t dd_stride, int64_t n_out, float *d_snr, int32_t *d_peak)
{
    BoxJob j{};
    j.dd = d_dd;
    j.dd_stride = dd_stride;
    j.n_out = n_out;
    j.snr = d_snr;
    j.peak = d_peak;
    j.n_dm = n_dm;
    // 16-byte row loads: aligned rows, and at least 4 samples
    j.vec_ok = (dd_stride % 4 == 0) && (((uintptr_t)d_dd & 15) == 0) && n_out >= 4;
    j.row_start = 0;
    return j;
}

namespace {

template <int NW, int LOOK>
amber_status launch_span_nw(bool pow2, bool vec, dim3 grid, dim3 block, size_t lds, hipStream_t stream, const BoxJob &one,
                    const BoxJob *d_jobs, int n_jobs, const WidthSet &ws)
{
    auto go = [&](auto kernel) -> amber_status {
        amber_status s = allow_lds(kernel, (int64_t)lds, "hipFuncSetAttribute(integrate_snr, span)");
        if (s == AMBER_OK) hipLaunchKernelGGL(kernel, grid, block, lds, stream, one, d_jobs, n_jobs, ws);
        return s;
    };
    if constexpr (LOOK == 1 || (NW > 7 && NW < 12))
        if (pow2) return vec ? go(span_snr_kernel<NW, true, true, LOOK>) : go(span_snr_kernel<NW, true, false, LOOK>);
    if constexpr (LOOK == 1 || NW % 4 == 0)
        return vec ? go(span_snr_kernel<NW, false, true, LOOK>) : go(span_snr_kernel<NW, false, false, LOOK>);
    return fail(AMBER_E_CONFIG, "no span kernel for %d widths", NW);
}

// The span kernel: at most 8 sliding widths up to kSpanMaxW per launch, or up
// to kSpanWideW in its wide form.
amber_status launch_span_snr(const BoxcarPlan &p, const BoxJob *single, const BoxJob *d_jobs, int n_jobs,
                             int64_t n_rows, const int32_t *widths, int n_widths, bool wide, bool vec,
                             hipStream_t stream)
{
    WidthSet ws{};
    bool pow2 = true;
    for (int k = 0; k < n_widths; ++k) {
        ws.w[k] = widths[k];
        pow2 = pow2 && widths[k] == (1 << k);
    }
    ws.n = n_widths;
    // the wide form is compiled for exact counts of powers of two, and for
    // counts up to 4, 8, 12 or 16 of any widths
    const int nw = !wide || pow2 ? n_widths : (n_widths + 3) / 4 * 4;
    const int threads = wide && p.threads > 512 ? 512 : p.threads;
    const int W = threads / kWave;
    const size_t lds = (size_t)W * (wide ? kSpanWideRing : kSpanRing) * 4 + (size_t)W * nw * (sizeof(SpanRes) + sizeof(double)) +
                       2 * (size_t)W * sizeof(long long);
    const BoxJob one = single ? *single : BoxJob{};
    const dim3 grid((unsigned)n_rows), block(threads);
    amber_status s = AMBER_OK;
#define SPAN(NW, LOOK) \
    case NW: s = launch_span_nw<NW, LOOK>(pow2, vec, grid, block, lds, stream, one, d_jobs, n_jobs, ws); break
    if (wide) {
        switch (nw) {
            SPAN(4, 4); SPAN(8, 4); SPAN(9, 4); SPAN(10, 4); SPAN(11, 4); SPAN(12, 4); SPAN(16, 4);
        default: return fail(AMBER_E_CONFIG, "span kernel (wide) takes 1 to 16 widths, got %d", n_widths);
        }
    } else {
        switch (nw) {
            SPAN(1, 1); SPAN(2, 1); SPAN(3, 1); SPAN(4, 1); SPAN(5, 1); SPAN(6, 1); SPAN(7, 1); SPAN(8, 1);
        default: return fail(AMBER_E_CONFIG, "span kernel takes 1 to 8 widths, got %d", n_widths);
        }
    }
#undef SPAN
    if (s != AMBER_OK) return s;
    AMBER_HIP(hipGetLastError(), "integrate_snr (span) launch");
    return AMBER_OK;
}

amber_status launch_dec_snr(const BoxcarPlan &p, const BoxJob &job, int64_t n_rows, const int32_t *factors, int n,
                            hipStream_t stream)
{
    WidthSet ws{};
    ws.n = n;
    for (int k = 0; k < n; ++k) {
        ws.w[k] = factors[k];
        ws.step[k] = k;
    }
    const int one = (int)(std::find(factors, factors + n, 1) - factors);
    if (one < n) {
        std::swap(ws.w[0], ws.w[one]);
        std::swap(ws.step[0], ws.step[one]);
    }
    const int threads = p.dec_threads ? p.dec_threads : (p.threads < 512 ? p.threads : 512), W = threads / kWave;
    const int nw = n <= 4 ? 4 : n <= 8 ? 8 : n <= 12 ? 12 : 16;
    const size_t lds = (size_t)W * (kDecChunk + AMBER_MAX_WIDTHS) * 4 + (size_t)W * (nw * sizeof(DecRes) + 4);
    auto go = [&](auto vec, auto any) -> amber_status {
        const auto kernel = job.vec_ok ? vec : any;
        amber_status s = allow_lds(kernel, (int64_t)lds, "hipFuncSetAttribute(downsample_snr)");
        if (s == AMBER_OK) hipLaunchKernelGGL(kernel, dim3((unsigned)n_rows), dim3(threads), lds, stream, job, ws);
        return s;
    };
    amber_status s = nw == 4    ? go(dec_snr_kernel<4, true>, dec_snr_kernel<4, false>)
                     : nw == 8  ? go(dec_snr_kernel<8, true>, dec_snr_kernel<8, false>)
                     : nw == 12 ? go(dec_snr_kernel<12, true>, dec_snr_kernel<12, false>)
                                : go(dec_snr_kernel<16, true>, dec_snr_kernel<16, false>);
    if (s != AMBER_OK) return s;
    AMBER_HIP(hipGetLastError(), "downsample_snr launch");
    return AMBER_OK;
}

}  // namespace

bool span_snr_applies(const int32_t *widths, int n_widths, int decimate, int64_t max_n_out)
{
    if (decimate || n_widths < 1 || n_widths > 8 || max_n_out >= ((int64_t)1 << 29)) return false;
    for (int k = 0; k < n_widths; ++k)
        if (widths[k] > kSpanMaxW) return false;
    return true;
}

bool span_wide_applies(const int32_t *widths, int n_widths, int decimate, int64_t max_n_out)
{
    if (decimate || n_widths < 1 || n_widths > 16 || max_n_out >= ((int64_t)1 << 29)) return false;
    for (int k = 0; k < n_widths; ++k)
        if (widths[k] > kSpanWideW) return false;
    return true;
}

amber_status launch_integrate_snr_jobs(const BoxcarPlan &p, const amber_tiles &t, const BoxJob *single,
                                       const BoxJob *d_jobs, int n_jobs, int64_t n_rows, const int32_t *widths,
                                       int n_widths, hipStream_t stream, int decimate, int all_vec,
                                       int64_t max_n_out)
{
    amber_status s = check_chunk(p);
    if (s != AMBER_OK) return s;
    if (n_rows > 0x7fffffff) return fail(AMBER_E_SHAPE, "too many rows (%lld)", (long long)n_rows);
    const int64_t longest = single ? single->n_out : max_n_out;
    const bool narrow = span_snr_applies(widths, n_widths, decimate, longest);
    // (one beam with more than 8 widths up to 64 takes passes of 8, below)
    const bool split = single && n_widths > 8 && *std::max_element(widths, widths + n_widths) <= kSpanMaxW;
    if (narrow || (!split && span_wide_applies(widths, n_widths, decimate, longest))) {
        const bool vec = single ? single->vec_ok != 0 : all_vec > 0;
        return launch_span_snr(p, single, d_jobs, n_jobs, n_rows, widths, n_widths, !narrow, vec, stream);
    }
    if (decimate && single && longest < ((int64_t)1 << 29))
        return launch_dec_snr(p, *single, n_rows, widths, n_widths, stream);
    // One beam with more than 8 series: passes of at most 8 (narrow span
    // kernels, as above, or for rows of 2^29 samples the chunk kernel, whose 16
    // running statistics would halve the resident work-groups).
    if (single && n_widths > 8) {
        for (int k0 = 0; k0 < n_widths; k0 += 8) {
            BoxJob j = *single;
            j.snr += (size_t)k0 * j.n_dm;
            if (j.peak) j.peak += (size_t)k0 * j.n_dm;
            amber_tiles tk = t;
            const int nk = n_widths - k0 < 8 ? n_widths - k0 : 8;
            for (int k = 0; k < nk; ++k) tk.boxcar_step[k] = t.boxcar_step[k0 + k];
            if ((s = launch_integrate_snr_jobs(p, tk, &j, nullptr, 1, n_rows, widths + k0, nk, stream, decimate, -1, j.n_out)) !=
                AMBER_OK)
                return s;
        }
        return AMBER_OK;
    }
    const WidthSet ws = make_widths(t, widths, n_widths, decimate);
    const int halo = halo_of(p);
    // the stats scratch reuses the prefix buffer after the last chunk
    int64_t lds = p.lds_bytes;
    const int64_t need = (int64_t)AMBER_MAX_WIDTHS * 16 * sizeof(Stat);
    if (lds < need) lds = need;
    const BoxJob one = single ? *single : BoxJob{};
    const dim3 grid((unsigned)n_rows);
    const int maxt = p.threads <= 256 ? 256 : (p.threads <= 512 ? 512 : 1024);
    auto go = [&](auto kernel) -> amber_status {
        amber_status st = allow_lds(kernel, lds, "hipFuncSetAttribute(integrate_snr)");
        if (st != AMBER_OK) return st;
        hipLaunchKernelGGL(kernel, grid, dim3(p.threads), (size_t)lds, stream, one, d_jobs, n_jobs, ws, p.chunk, halo);
        return AMBER_OK;
    };
    if (n_widths <= 4)
        s = maxt == 256 ? go(integrate_snr_kernel<4, 256>)
                        : (maxt == 512 ? go(integrate_snr_kernel<4, 512>) : go(integrate_snr_kernel<4, 1024>));
    else if (n_widths <= 8)
        s = maxt == 256 ? go(integrate_snr_kernel<8, 256>)
                        : (maxt == 512 ? go(integrate_snr_kernel<8, 512>) : go(integrate_snr_kernel<8, 1024>));
    else
        s = maxt == 256 ? go(integrate_snr_kernel<16, 256>)
                        : (maxt == 512 ? go(integrate_snr_kernel<16, 512>) : go(integrate_snr_kernel<16, 1024>));
    if (s != AMBER_OK) return s;
    AMBER_HIP(hipGetLastError(), "integrate_snr launch");
    return AMBER_OK;
}

amber_status launch_integrate_snr(const BoxcarPlan &p, const amber_tiles &t, const int32_t *d_dd, int n_dm,
                                  int64_t dd_stride, int64_t n_out, const int32_t *widths, int n_widths,
                                  float *d_snr, int32_t *d_peak, hipStream_t stream, int decimate)
{
    const BoxJob j = make_box_job(d_dd, n_dm, dd_stride, n_out, d_snr, d_peak);
    return launch_integrate_snr_jobs(p, t, &j, nullptr, 1, n_dm, widths, n_widths, stream, decimate);
}

amber_status launch_integrate(const BoxcarPlan &p, const amber_tiles &t, const int32_t *d_dd, int n_dm,
                              int64_t dd_stride, int64_t n_out, const int32_t *widths, int n_widths, int32_t *d_box,
                              int64_t box_stride, hipStream_t stream, int decimate)
{
    amber_status s = check_chunk(p);
    if (s != AMBER_OK) return s;
    const WidthSet ws = make_widths(t, widths, n_widths, decimate);
    const int halo = halo_of(p);
    const int outs = p.chunk - halo;
    const int64_t n_chunks = (n_out + outs - 1) / outs;
    const int vec_ok = (dd_stride % 4 == 0) && (((uintptr_t)d_dd & 15) == 0);
    if ((s = allow_lds(integrate_kernel, p.lds_bytes, "hipFuncSetAttribute(integrate)")) != AMBER_OK) return s;
    hipLaunchKernelGGL(integrate_kernel, dim3((unsigned)n_chunks, n_dm), dim3(p.threads), (size_t)p.lds_bytes, stream,
                       d_dd, n_dm, dd_stride, n_out, ws, p.chunk, halo, vec_ok, d_box, box_stride);
    AMBER_HIP(hipGetLastError(), "integrate launch");
    return AMBER_OK;
}

amber_status launch_snr(const BoxcarPlan &p, const amber_tiles &t, const int32_t *d_box, int n_dm, int64_t box_stride,
                        int64_t n_out, const int32_t *widths, int n_widths, float *d_snr, int32_t *d_peak,
                        hipStream_t stream)
{
    const WidthSet ws = make_widths(t, widths, n_widths, 0);
    const bool vec = box_stride % 4 == 0 && ((uintptr_t)d_box & 15) == 0;
    hipLaunchKernelGGL(vec ? snr_kernel<true> : snr_kernel<false>, dim3(n_dm, n_widths), dim3(p.threads), 0, stream,
                       d_box, n_dm, box_stride, n_out, ws, d_snr, d_peak);
    AMBER_HIP(hipGetLastError(), "snr launch");
    return AMBER_OK;
}

}  // namespace amber
