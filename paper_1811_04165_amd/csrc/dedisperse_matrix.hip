// Brute-force dedispersion on the matrix cores.
//
//   dd[i][t] = sum over c of in[c][t + delay[i][c]]
//
// Neighbouring channels move almost alike: over 32 consecutive trials and 64
// consecutive channels, delay[i][c] is a shift of the trial (that of the
// group's middle channel, less its shift at the first trial) plus a small
// remainder r in 0 .. S - 1 that depends on trial and channel, once each
// channel's window starts at a sample of its own.  With the channels as the
// contraction index, the sums of the group are then S small products
//
//   G[i][u] = sum over s < S, c of [r(i, c) = s] * x[c][start(c) + u + s]
//
// of a 0/1 matrix (trials x channels) with the samples (channels x columns),
// and dd[i][t] gains G[i][t + shift(i)].  One v_mfma_i32_32x32x32_i8 does 32
// trials x 32 channels x 32 columns for one s; the shift is the address at
// which the 32 x 32 results are added to the work-group's sums in LDS.
// Everything is integer and exact for every table: S is taken from the table
// on the device, and a group with a large S is cut into passes of NS remainders.
// Which channels make a group is free: where those that come together do not
// move alike (a band listed in another order than by frequency), the work-group
// sorts them by how far they move and forms groups anew.  A group that needs
// more than kRoughS remainders even so is summed directly.
//
// What bounds it: per 32 channels x 64 columns a wavefront issues 2 NS products
// (35 clocks of a SIMD each), 2 KiB of staging writes, NS + 1 reads and 16
// 64-bit additions (4.3, 4.3 and 6.2 LDS clocks per wavefront instruction), so
// matrix cores, LDS and the byte shuffles of the staging are each busy a third
// to half of the time, and the latencies between them show: two wavefronts per
// SIMD are all that the 0/1 matrices' registers allow.  Of the 365-415 us that
// 1536 channels x 2048 trials x 12208 samples take (105 T additions/s; the
// vector kernel: 1040 us, 37 T), the products alone take 70, the staging 75,
// the additions 50, reading the delays and finding the remainders 40, the
// passes' starts 50.
#include "internal.h"

#include <algorithm>
#include <cstdlib>
#include <type_traits>
#include <vector>

namespace amber {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) int32_t lds_i;
typedef __attribute__((address_space(3))) uint32_t lds_u;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) uint64_t lds_u64;
typedef __attribute__((address_space(3))) const v4i lds_v4;
typedef __attribute__((address_space(3))) v4i lds_w4;
typedef int v2i __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const v2i lds_v2;
typedef __attribute__((address_space(3))) v2i lds_w2;

constexpr int kRows = kMatRows;  // trials per work-group: the rows of a product
constexpr int kChunk = 64;       // columns staged at a time
constexpr int kGroup = 32;       // channels per group: the depth of a product
constexpr int kRoughS = 128;     // groups with more remainders are summed directly
constexpr int kWindow = 2048;    // channels that are sorted together, at most
constexpr int kBins = 1024;      // by distance (omax is below 800 where 128 columns fit)
// LDS of a wavefront: a ring of two chunks of columns x 32 channels, 16
// channels of one column per 16-byte line, the columns of 16 channels in a
// plane of their own, even columns before odd ones (a group's delays pass
// through the same place first); then the window starts [32], the trial
// shifts [32] and the channels' smallest offsets, packed [16].
constexpr int kPlane = 2 * kChunk * 16;
constexpr int kOdd = kPlane / 2;
constexpr int kLine = 4 * kGroup + 16;  // bytes of a trial's delays, padded against bank conflicts
constexpr int kStart = kRows * kLine, kShift = kStart + 4 * kGroup, kLow = kShift + 4 * kRows;
constexpr int kWaveLds = 5120;  // a multiple of kOdd: ring addresses wrap within their low bits
// Sorted channels: 16 bits each, 256 in each wavefront's part between the ring
// and the tables (the delays of sorted channels are staged without padding); in
// wavefront 0's after the tables, a bit for each group that is set aside.
constexpr int kOrder = 2 * kPlane, kAside = kLow + 64;
static_assert(kAside + 32 <= kWaveLds && kWaveLds % kOdd == 0, "tables fit");
static_assert(kOrder + 2 * kWindow / kMatWaves <= kStart && 4 * kBins <= kOrder, "the ring and the order fit");
static_assert(kMatWaveLds == kWaveLds, "planner and kernel agree");

// LDS by byte offset.
template <typename T>
__device__ __forceinline__ T *lds(int offset)
{
    return (T *)(uintptr_t)(uint32_t)offset;
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t range_rsrc(const void *p, uint32_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)n, 0x00020000);
}

template <int CTRL>
__device__ __forceinline__ int dpp(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}

__device__ __forceinline__ int pk_min(int a, int b)
{
    const s16x2 r = __builtin_elementwise_min(__builtin_bit_cast(s16x2, a), __builtin_bit_cast(s16x2, b));
    return __builtin_bit_cast(int, r);
}
__device__ __forceinline__ int pk_max(int a, int b)
{
    const s16x2 r = __builtin_elementwise_max(__builtin_bit_cast(s16x2, a), __builtin_bit_cast(s16x2, b));
    return __builtin_bit_cast(int, r);
}
__device__ __forceinline__ int pk_sub(int a, int b)
{
    const s16x2 r = __builtin_bit_cast(s16x2, a) - __builtin_bit_cast(s16x2, b);
    return __builtin_bit_cast(int, r);
}
__device__ __forceinline__ int pk_min_u(int a, int b)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 r = __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b));
    return __builtin_bit_cast(int, r);
}

// One step of a packed minimum over lanes that also spreads the N registers of
// t over them: the N / 2 left hold, in lanes with `upper` clear, the minimum
// of registers 0, 2, .. with the partner lanes', in the others that of 1, 3, ..
template <int N, int CTRL, int M>
__device__ __forceinline__ void min_step(int (&t)[M], bool upper)
{
#pragma unroll
    for (int m = 0; m < N / 2; ++m) {
        const int keep = upper ? t[2 * m + 1] : t[2 * m], give = upper ? t[2 * m] : t[2 * m + 1];
        t[m] = pk_min(keep, dpp<CTRL>(give));
    }
}

// Maximum over the wavefront.
__device__ __forceinline__ int wave_max(int v)
{
    v = max(v, dpp<0xb1>(v));
    v = max(v, dpp<0x4e>(v));
    v = max(v, dpp<0x141>(v));
    v = max(v, dpp<0x140>(v));
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// What a wavefront knows of its work-group's tile.
struct Tile {
    __amdgpu_buffer_rsrc_t rd;   // delay rows of the tile's trials
    const int32_t *delays;
    const uint8_t *in;
    const uint8_t *keep;
    int64_t in_stride, in_bytes, t0;
    int n_chan, rows, omax;
    int T, cols;                 // columns of the tile, columns below n_out
    int acc, pitch;              // the sums in LDS: byte offset of row 0, dwords from row to row
    int ring;                    // LDS byte offset of the wavefront's part
    int lane;
    // The channels at hand: count of them, in their own order, or (ORDER, in the
    // functions below) listed in LDS, the task's from order on, as offsets from
    // channel row0.
    int count, order, row0;
};

// The remainders of the 32 channels from c0 on (of those at hand): lane l holds those of trial
// l & 31 and of the 16 channels 16 (l >> 5) + j, packed in 16-bit pairs
// (0x7fff for channels that do not count).
struct Rem {
    int p[8];
    int S;       // remainders are below S (wave-uniform)
    int most;    // the largest shift of a trial (wave-uniform)
    bool aside;  // set aside for sorting (wave-uniform; not with ORDER)
    int first;   // where the window of the channel at the loads' base starts (wave-uniform)
};

template <int NS, bool ORDER>
__device__ __forceinline__ void remainders(const Tile &k, int c0, Rem &r)
{
    const int lane = k.lane, row = min(lane & 31, k.rows - 1), h = lane >> 5;
    const int nv = min(kGroup, k.count - c0);
    const int pitch = 4 * k.n_chan;
    int line = kLine;
    // lane j's channel
    int channel = c0 + (lane & 31);
    // The group's delays go through LDS: loaded as whole pieces of rows (8
    // lanes of 16 bytes per trial; the last row's may end past the table, where
    // each dword counts by itself) and read back by trial.
    if (!ORDER) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = 8 * q + (lane >> 3), piece = lane & 7;
            const v4i x = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                                                      k.rd, min(i, k.rows - 1) * pitch + 4 * c0 + 16 * piece, 0, 0));
            *lds<lds_w4>(k.ring + i * kLine + 16 * piece) = x;
        }
    } else {
        line = 4 * kGroup;
        channel = k.row0 + *lds<lds_u16>(k.order + 2 * (lane & 31));
        int x[kRows / 2];
#pragma unroll
        for (int q = 0; q < kRows / 2; ++q)
            x[q] = (int)__builtin_amdgcn_raw_buffer_load_b32(k.rd, min(2 * q + h, k.rows - 1) * pitch + 4 * channel, 0, 0);
#pragma unroll
        for (int q = 0; q < kRows / 2; ++q) *lds<lds_i>(k.ring + (2 * q + h) * line + 4 * (lane & 31)) = x[q];
    }
    __builtin_amdgcn_wave_barrier();
    // the shift is that of the middle channel (one outside the range that the
    // table's summary allows is clamped: sums may go wrong then, addresses may
    // not)
    const int mid = 4 * (nv >> 1);
    const int s0 = *lds<lds_i>(k.ring + mid), si = *lds<lds_i>(k.ring + row * line + mid);
    const int shift = min(max(si - s0, 0), k.omax) & ~1;  // even: columns are added in pairs
    r.most = uniform(wave_max(shift));
    int pair[8];  // offsets less the shift, two channels a dword
    const int shift2 = (shift & 0xffff) | (shift << 16);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int o = k.ring + 64 * h + 16 * q;
        const v4i d = *lds<lds_v4>(o + row * line) - *lds<lds_v4>(o);
        pair[2 * q] = pk_sub((int)__builtin_amdgcn_perm((uint32_t)d[1], (uint32_t)d[0], 0x05040100u), shift2);
        pair[2 * q + 1] = pk_sub((int)__builtin_amdgcn_perm((uint32_t)d[3], (uint32_t)d[2], 0x05040100u), shift2);
    }
    // Each channel's smallest over the trials: lane l of a half ends up with
    // that of pair m(l); every step halves the number of registers.
    const int mine = lane & 31;
    int t[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const auto x = __builtin_amdgcn_permlane16_swap(pair[2 * m], pair[2 * m + 1], false, false);
        t[m] = pk_min((int)x[0], (int)x[1]);
    }
    min_step<4, 0x128>(t, (mine & 8) != 0);  // row_ror:8
    min_step<2, 0x141>(t, (mine & 4) != 0);  // row_half_mirror
    t[0] = pk_min(t[0], dpp<0x4e>(t[0]));    // quad_perm [2,3,0,1]
    t[0] = pk_min(t[0], dpp<0xb1>(t[0]));    // quad_perm [1,0,3,2]
    const int m = ((mine >> 4) & 1) | ((mine >> 2) & 2) | (mine & 4);
    const int c2 = 16 * h + 2 * m;  // its first channel
    const v2i start = *lds<lds_v2>(k.ring + 4 * c2) + v2i{(int)(short)t[0], t[0] >> 16};
    r.first = uniform(start.x);  // (lane 0 has channel 0)
    *lds<lds_w2>(k.ring + kStart + 4 * c2) = start;
    if (ORDER) {
        const uint32_t at = (uint32_t)__builtin_amdgcn_ballot_w64(channel == k.row0) & (0xffffffffu >> (kGroup - nv));
        r.first = at ? uniform(*lds<lds_i>(k.ring + kStart + 4 * __builtin_ctz(at))) : 0;
    }
    *lds<lds_i>(k.ring + kLow + 32 * h + 4 * m) = t[0];
    if (lane < 32) *lds<lds_i>(k.ring + kShift + 4 * lane) = shift;
    __builtin_amdgcn_wave_barrier();
    int worst = 0;
    const bool all = nv == kGroup && !k.keep;
    uint32_t valid = 0xffffu;
    if (!all) {
        const uint32_t ok =
            (uint32_t)__builtin_amdgcn_ballot_w64((lane & 31) < nv && (!k.keep || k.keep[channel] != 0));
        valid = (ok >> (16 * h)) & 0xffffu;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const v4i lo = *lds<lds_v4>(k.ring + kLow + 32 * h + 16 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int p = 4 * q + e;
            int v = pk_sub(pair[p], lo[e]);
            if (!all) {
                // channels that do not count: no remainder for S, none to match
                const int ok = ((valid >> (2 * p)) & 1u ? 0xffff : 0) | ((valid >> (2 * p + 1)) & 1u ? (int)0xffff0000 : 0);
                worst = pk_max(worst, v & ok);
                v = (v & ok) | (0x7fff7fff & ~ok);
            } else {
                worst = pk_max(worst, v);
            }
            r.p[p] = v;
        }
    }
    r.S = uniform(wave_max(max((int)(short)worst, worst >> 16))) + 1;
    r.aside = false;
    if (!ORDER && r.S > 2 * NS) {
        // Sorting helps a group that goes back and forth over the tile's last
        // trial (lanes 31 and 63), or sweeps over more than its share of the
        // band: a group in order of frequency at the narrow end has 6.4 times
        // its share, at most, of a band whose top is 4 times its bottom.
        int way = 0, low = pair[0], high = pair[0];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            low = pk_min(low, pair[p]);
            high = pk_max(high, pair[p]);
            const int in = pair[p] >> 16, out = p < 7 ? (int)(short)pair[p < 7 ? p + 1 : 7] : in;
            way += abs(in - (int)(short)pair[p]) + abs(out - in);
        }
        const int lo = min((int)(short)low, low >> 16), hi = max((int)(short)high, high >> 16);
        const int join = abs((int)(short)__builtin_amdgcn_readlane(pair[0], 63) - (__builtin_amdgcn_readlane(pair[7], 31) >> 16));
        const int ways = __builtin_amdgcn_readlane(way, 31) + __builtin_amdgcn_readlane(way, 63) + join;
        const int range = max(__builtin_amdgcn_readlane(hi, 31), __builtin_amdgcn_readlane(hi, 63)) -
                          min(__builtin_amdgcn_readlane(lo, 31), __builtin_amdgcn_readlane(lo, 63));
        r.aside = ways > 2 * range || 2 * (r.S - 2) * k.n_chan > 13 * kGroup * k.omax;
    }
}

// The staging of one chunk of 64 columns: lane (q, i) = (lane >> 3, lane & 7)
// takes columns 8 i .. 8 i + 7 of the 4 channels of quad q.  The vector cache
// serves four lanes per clock where they share a line and their addresses are
// whole dwords, whatever their width, so each lane loads the two dwords that
// end its columns; the dword before them is its neighbour's last, or the
// chunk's before.
struct Stage {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t off[4];      // byte offsets of the next chunk's loads, plus the misalignment
    uint32_t before[4];   // in lane i = 0: the dword before the lane's two
    int at;               // ring address (slot 0) of the first columns the lane writes
};

struct Chunk {
    v2i w[4];
};

template <bool ORDER>
__device__ __forceinline__ void stage_begin(const Tile &k, int c0, int skip, int m, Stage &s)
{
    const int q = k.lane >> 3, i = k.lane & 7;
    const int64_t from = (int64_t)(ORDER ? k.row0 : c0) * k.in_stride;
    const int64_t rest = k.in_bytes - from;
    s.rs = range_rsrc(k.in + from, (uint32_t)(rest < 0xfffffff0ll ? rest : 0xfffffff0ll));
    const v4i st = *lds<lds_v4>(k.ring + kStart + 16 * q);
    v4i channel = {4 * q, 4 * q + 1, 4 * q + 2, 4 * q + 3};  // from the base
    if (ORDER) {
        const v2i two = *lds<lds_v2>(k.order + 8 * q);
        channel = v4i{two.x & 0xffff, (int)((uint32_t)two.x >> 16), two.y & 0xffff, (int)((uint32_t)two.y >> 16)};
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        // columns before the first row's start wrap to offsets out of range
        // and read zeros (no sum needs them)
        const uint32_t o = (uint32_t)channel[j] * (uint32_t)k.in_stride +
                           (uint32_t)((int)k.t0 + st[j] + skip + kChunk * m);
        s.before[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(s.rs, o & ~3u, 0, 0);
        s.off[j] = o + 4u + 8u * (uint32_t)i;
    }
    s.at = (k.ring + (q >> 2) * kPlane + 4 * (q & 3) + 64 * i) ^ (i & 4 ? 16 : 0);
}

// Loads the next chunk.
__device__ __forceinline__ void stage_load(Stage &s, Chunk &c)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c.w[j] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(s.rs, s.off[j] & ~3u, 0, 0));
        s.off[j] += kChunk;
    }
}

// Writes a chunk into the ring's slot at slot_bytes: per column a dword of 4
// channels, as signed bytes (sample - 128).  32 lanes write at once and have
// to cover 32 banks: lanes i and i + 4 hold columns 32 apart, which lie in the
// same banks, so that these take the columns of each group of four in another
// order (2, 3, 0, 1).
__device__ __forceinline__ void stage_write(int lane, Stage &s, int slot_bytes, const Chunk &c)
{
    // v_perm selectors: the first and last two columns of two channels
    const uint32_t front = lane & 4 ? 0x07030602u : 0x05010400u, back = lane & 4 ? 0x05010400u : 0x07030602u;
    uint32_t d[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t last = (uint32_t)c.w[j].y;
        // row_shr:1, but the first of 8 lanes has the last of the chunk
        // before, which row_half_mirror brought there
        const uint32_t shr = (uint32_t)__builtin_amdgcn_mov_dpp((int)last, 0x111, 0xf, 0xf, true);
        const uint32_t left = (lane & 7) == 0 ? s.before[j] : shr;
        s.before[j] = (uint32_t)__builtin_amdgcn_mov_dpp((int)last, 0x141, 0xf, 0xf, true);
        // (of the shift, the low two bits count)
        d[j][0] = __builtin_amdgcn_alignbyte((uint32_t)c.w[j].x, left, s.off[j]) ^ 0x80808080u;
        d[j][1] = __builtin_amdgcn_alignbyte(last, (uint32_t)c.w[j].x, s.off[j]) ^ 0x80808080u;
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const uint32_t a01 = __builtin_amdgcn_perm(d[1][g], d[0][g], front);
        const uint32_t a23 = __builtin_amdgcn_perm(d[3][g], d[2][g], front);
        const uint32_t b01 = __builtin_amdgcn_perm(d[1][g], d[0][g], back);
        const uint32_t b23 = __builtin_amdgcn_perm(d[3][g], d[2][g], back);
        lds_u *to = lds<lds_u>(s.at + slot_bytes) + g * 8;
        lds_u *up = lds<lds_u>((s.at ^ 16) + slot_bytes) + g * 8;
        to[0] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
        to[kOdd / 4] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
        up[0] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
        up[kOdd / 4] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
    }
}

// A product's sums start here, so that they are never negative (32 channels of
// -128 * (sample - 128)): two neighbouring columns can then be added as one
// 64-bit number.
constexpr int kStartSum = 128 * 127 * kGroup;

// Adds a chunk's results to the sums.  Lane l holds columns 2 (l & 31) and
// 2 (l & 31) + 1 of the chunk (even and odd) and rows (v & 3) + 8 (v >> 2) +
// 4 (l >> 5); at[v] is the LDS byte address of that row's column 2 (l & 31)
// for this lane, moved on to the next chunk.  Two columns go in one 64-bit
// addition (6.2 clocks of the LDS against twice 4.3).  Columns that fall
// outside a row's T fall into the space between the rows (a select per
// addition cost as much as the products: two of five chunks have such
// columns).
__device__ __forceinline__ void add_chunk(const v16i &even, const v16i &odd, int (&at)[16])
{
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const uint64_t x = (uint32_t)even[v] | ((uint64_t)(uint32_t)odd[v] << 32);
        __hip_atomic_fetch_add(lds<lds_u64>(at[v]), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        at[v] += 4 * kChunk;
    }
}

// How many columns early (0 or 4) a pass takes a group whose first channel's
// window starts `first` samples off the buffer's begin.  A load of two dwords
// whose first wraps out of range counts as out of range as a whole, also where
// its second begins the row; 4 columns earlier no load is of that kind.  (Past
// the end each dword counts by itself.)
__device__ __forceinline__ int columns_early(int first) { return first < 0 ? (first + 4) & 4 : 0; }

// One pass: chunks [j0, j1) of 64 columns, `early` columns before their place,
// remainders skip .. skip + NS - 1 in r.  A chunk's even and odd columns are
// two products: column 2 n + phi with remainder s is sample column 2 n + w, w =
// phi + s, so one read serves both.
template <int NS, bool ORDER>
__device__ __forceinline__ void pass(const Tile &k, const Rem &r, int c0, int skip, int early, int j0, int j1)
{
    const int lane = k.lane, h = lane >> 5, n = lane & 31;
    if (j0 >= j1) return;
    Stage st;
    stage_begin<ORDER>(k, c0, skip - early, j0, st);
    Chunk w, w1;
    stage_load(st, w);
    stage_load(st, w1);

    // The 0/1 matrices: byte c of a lane's 16 is -128 (0x80) where the
    // remainder is s, else 0.  z = remainder ^ s is 0 there and at most 0x7f
    // elsewhere, so 0x80 - z sets bit 7 only there and borrows from no
    // neighbour.
    v4i W[NS];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int s2 = skip | (skip << 16);
        const int lo = pk_min_u(pk_sub(r.p[2 * q], s2), 0x007f007f);
        const int hi = pk_min_u(pk_sub(r.p[2 * q + 1], s2), 0x007f007f);
        const uint32_t rb = __builtin_amdgcn_perm((uint32_t)hi, (uint32_t)lo, 0x06040200u);
#pragma unroll
        for (int s = 0; s < NS; ++s) W[s][q] = (int)((0x80808080u - (rb ^ (0x01010101u * (uint32_t)s))) & 0x80808080u);
    }

    // where the results go
    int at[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const v4i sh = *lds<lds_v4>(k.ring + kShift + 4 * (8 * g + 4 * h));
#pragma unroll
        for (int e = 0; e < 4; ++e)
            at[4 * g + e] = k.acc + 4 * ((8 * g + 4 * h + e) * k.pitch + 2 * n - sh[e] - early + kChunk * j0);
    }
    constexpr int kSlot = kOdd / 2;  // the ring's second slot follows the first
    stage_write(lane, st, 0, w);
    stage_load(st, w);
    stage_write(lane, st, kSlot, w1);

    v16i start;
#pragma unroll
    for (int v = 0; v < 16; ++v) start[v] = kStartSum;
    asm volatile("" : "+v"(start));  // held in registers
    v4i B[NS + 1];  // sample columns w of a chunk
    const int plane = k.ring + h * kPlane;
    auto read = [&](int slot) {
        int line = 16 * (lane & 31) + slot;
        asm volatile("" : "+v"(line));  // (the addresses are not worth registers all along)
#pragma unroll
        for (int x = 0; x <= NS; ++x) {
            // columns past the ring's end are at its start
            const int a = x < 2 ? plane + line : plane | ((line + 16 * (x >> 1)) & (kOdd - 1));
            B[x] = *lds<lds_v4>(a + (x & 1) * kOdd);
        }
    };
    read(0);
    int slot = 0;
    for (int j = j0; j < j1; ++j) {
        v16i g0 = start, g1 = start;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x <= NS; ++x) {
            if (x < NS) g0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(W[x], B[x], g0, 0, 0, 0);
            if (x > 0) g1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(W[x - 1], B[x], g1, 0, 0, 0);
        }
        // The chunk after next replaces this one, whose reads came before (a
        // wavefront's LDS operations keep their order).
        stage_write(lane, st, slot, w);
        stage_load(st, w);
        __builtin_amdgcn_sched_barrier(0);
        // the next chunk's reads go ahead of this one's additions, which would
        // keep them waiting
        slot ^= kSlot;
        read(slot);
        __builtin_amdgcn_sched_barrier(0);
        add_chunk(g0, g1, at);
    }
}

// A group whose channels do not move alike: every trial and channel on its
// own, 512 columns at a time (8 per lane), four trials at once.
template <bool ORDER>
__device__ __forceinline__ void direct_group(const Tile &k, int c0)
{
    const int left = min(kGroup, k.count - c0), base = ORDER ? k.row0 : c0;
    const int64_t from = (int64_t)base * k.in_stride;
    const int64_t rest = k.in_bytes - from;
    const __amdgpu_buffer_rsrc_t rs = range_rsrc(k.in + from, (uint32_t)(rest < 0xfffffff0ll ? rest : 0xfffffff0ll));
    for (int t = 0; t < k.cols; t += 512) {
        for (int i = 0; i < k.rows; i += 4) {
            uint32_t lo[4][2] = {}, hi[4][2] = {};
            int count = 0;
            for (int j = 0; j < left; ++j) {
                const int c = ORDER ? uniform(*lds<lds_u16>(k.order + 2 * j)) : j;  // from the base
                if (k.keep && k.keep[base + c] == 0) continue;
                ++count;
                const int d0 = uniform(k.delays[base + c]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int d = uniform(k.delays[(size_t)min(i + e, k.rows - 1) * k.n_chan + base + c]);
                    const int o = d0 + min(max(d - d0, 0), k.omax);
                    const uint32_t x = (uint32_t)c * (uint32_t)k.in_stride + (uint32_t)((int)k.t0 + t + o + 8 * k.lane);
                    const auto v = __builtin_amdgcn_raw_buffer_load_b96(rs, x & ~3u, 0, 0);
                    const uint32_t a = __builtin_amdgcn_alignbyte(v[1], v[0], x & 3u);
                    const uint32_t b = __builtin_amdgcn_alignbyte(v[2], v[1], x & 3u);
                    lo[e][0] += a & 0x00ff00ffu;
                    hi[e][0] += (a >> 8) & 0x00ff00ffu;
                    lo[e][1] += b & 0x00ff00ffu;
                    hi[e][1] += (b >> 8) & 0x00ff00ffu;
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (i + e >= k.rows) break;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const uint32_t pair = (q & 1) ? hi[e][q >> 2] : lo[e][q >> 2];
                    const int v = (int)((q & 2) ? pair >> 16 : pair & 0xffffu);
                    const int u = t + 8 * k.lane + q;
                    if (u < k.T)
                        __hip_atomic_fetch_add(lds<lds_i>(k.acc + 4 * ((i + e) * k.pitch + u)),
                                               kStartSum - 128 * (v - 128 * count), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
    }
}

// What a work-group keeps in LDS beside the wavefronts' parts and the sums, by
// byte offset from `next`: the next task, zapped jobs' kept channels, the
// passes made, and the number of groups set aside (from bit 16 on) and of the
// passes that they would have taken.
constexpr int kKept = 4, kPasses = 8, kAsidePasses = 12;

// Sorts the channels of the groups set aside among those from k.row0 on (up to
// `window`) by how far they move over the tile's trials, where the groups formed
// of them then take at least a fifth fewer passes; else they keep their order.
// Leaves their list in LDS and their number in k.count.  By the whole
// work-group, with barriers.
__device__ __forceinline__ void regroup(Tile &k, int base, int next, int window, int ns)
{
    constexpr int kThreads = 64 * kMatWaves, kEach = kWindow / kThreads, kPer = kBins / 64;
    const int tid = threadIdx.x, end = min(k.n_chan, k.row0 + window);
    const auto slot = [&](int rank) { return lds<lds_u16>(base + (rank >> 8) * kWaveLds + kOrder + 2 * (rank & 255)); };
    // this work-item's channels: their bins, or -1
    int bin[kEach];
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
        const int c = k.row0 + q * kThreads + tid;
        bin[q] = -1;
        if (c < end && ((*lds<lds_u>(base + kAside + 4 * (c >> 10)) >> ((c >> 5) & 31)) & 1u) && (!k.keep || k.keep[c] != 0))
            bin[q] = min(max(k.delays[(size_t)(k.rows - 1) * k.n_chan + c] - k.delays[c], 0), kBins - 1);
    }
    for (int b = tid; b < kBins / 4; b += kThreads) *lds<lds_w4>(base + 16 * b) = v4i{0, 0, 0, 0};
    if (tid == 0) *lds<lds_i>(next) = kMatWaves;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kEach; ++q)
        if (bin[q] >= 0)
            __hip_atomic_fetch_add(lds<lds_i>(base + 4 * bin[q]), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    // the bins' first ranks, by every wavefront (wavefront 0's are kept)
    int n[kPer], sum = 0, low = kBins, high = -1;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        n[e] = *lds<lds_i>(base + 4 * (kPer * k.lane + e));
        low = n[e] != 0 && low == kBins ? kPer * k.lane + e : low;
        high = n[e] != 0 ? kPer * k.lane + e : high;
        sum += n[e];
    }
    int before = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(before, off, 64);
        if (k.lane >= off) before += y;
    }
    const int total = __builtin_amdgcn_readlane(before, 63);
    before -= sum;
    // passes of sorted groups, at most: together they span the bins once
    const int groups = (total + kGroup - 1) / kGroup;
    const int passes = groups + (wave_max(high) + wave_max(-low) + 2 * groups) / ns;
    // those of the window's groups as they are: the mean of the ones looked at
    int here = 0;
    for (int w = k.row0 >> 10; 1024 * w < end; ++w) {
        const int from = max(k.row0 / kGroup - 32 * w, 0), to = min((end + kGroup - 1) / kGroup - 32 * w, 32);
        here += __builtin_popcount(*lds<lds_u>(base + kAside + 4 * w) >> from << from & 0xffffffffu >> (32 - to));
    }
    const int seen = *lds<lds_i>(next + kAsidePasses);
    const bool sort = 5 * passes * (seen >> 16) < 4 * (seen & 0xffff) * here;
    __syncthreads();
    if (sort) {
        if (tid < 64) {
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                *lds<lds_i>(base + 4 * (kPer * k.lane + e)) = before;
                before += n[e];
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kEach; ++q)
            if (bin[q] >= 0)
                *slot(__hip_atomic_fetch_add(lds<lds_i>(base + 4 * bin[q]), 1, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP)) = (uint16_t)(q * kThreads + tid);
        k.count = total;
    } else {
        // whole groups one after the other
        int rank = 0;
        for (int c = k.row0; c < end; c += kGroup) {
            if (!((*lds<lds_u>(base + kAside + 4 * (c >> 10)) >> ((c >> 5) & 31)) & 1u)) continue;
            const int m = min(kGroup, end - c);
            if (tid < m) *slot(rank + tid) = (uint16_t)(c - k.row0 + tid);
            rank += m;
        }
        k.count = rank;
    }
    // the last group's places that no channel has
    if (tid < (-k.count & (kGroup - 1))) *slot(k.count + tid) = 0;
    __syncthreads();
}

// A wavefront's tasks: groups of 32 channels, each in `parts` column ranges,
// taken by the wavefronts as they come free.  First the channels as they come;
// groups of more than two passes that sorting may help are set aside, and their
// channels come again after that (ORDER).
template <int NS, bool ORDER>
__device__ __forceinline__ void tasks(Tile &k, int base, int next, int parts, int wave)
{
    const auto add_to = [&](int what, int n) {
        __hip_atomic_fetch_add(lds<lds_i>(next + what), n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    const int n_tasks = (k.count + kGroup - 1) / kGroup * parts;
    for (int task = wave; task < n_tasks;) {
        // what depends on the lane is worked out per task: hoisted out of this
        // loop it would not fit the registers
        asm volatile("" : "+v"(k.lane));
        const int sub = task / parts, part = task - sub * parts;
        const int c0 = sub * kGroup;
        if (ORDER) {
            k.order = base + (c0 >> 8) * kWaveLds + kOrder + 2 * (c0 & 255);
        } else if (k.keep && part == 0) {
            const int c = c0 + k.lane;
            const uint64_t m = __builtin_amdgcn_ballot_w64(k.lane < kGroup && c < k.n_chan && k.keep[min(c, k.n_chan - 1)] != 0);
            if (k.lane == 0) add_to(kKept, (int)__builtin_popcountll(m));
        }
        Rem r;
        remainders<NS, ORDER>(k, c0, r);
        if (!ORDER && r.aside) {
            if (part == 0 && k.lane == 0) {
                __hip_atomic_fetch_or(lds<lds_u>(base + kAside + 4 * (sub >> 5)), 1u << (sub & 31), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
                add_to(kAsidePasses, 0x10000 + min((r.S + NS - 1) / NS, 64));
            }
        } else {
            if (part == 0 && k.lane == 0) add_to(kPasses, r.S > kRoughS ? 1 : (r.S + NS - 1) / NS);
            if (r.S > kRoughS) {
                if (part == 0) direct_group<ORDER>(k, c0);
            } else {
                const int first = (int)k.t0 + r.first;
                for (int skip = 0; skip < r.S; skip += NS) {
                    const int early = columns_early(first + skip);
                    const int chunks = (k.cols + r.most + early + kChunk - 1) / kChunk;
                    pass<NS, ORDER>(k, r, c0, skip, early, chunks * part / parts, chunks * (part + 1) / parts);
                }
            }
        }
        int t = 0;
        if (k.lane == 0)
            t = __hip_atomic_fetch_add(lds<lds_i>(next), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        task = uniform(t);
    }
}

template <int NS>
__global__ __launch_bounds__(64 * kMatWaves) __attribute__((amdgpu_waves_per_eu(kMatWaves / 4, kMatWaves / 4)))
void dedisperse_matrix_kernel(DedispJob single, const DedispJob *__restrict__ jobs, int n_jobs, int T, int remap)
{
    extern __shared__ v4i lds_raw[];
    int block = blockIdx.x;
    DedispJob job = single;
    if (jobs) {
        int j = 0;
        while (j + 1 < n_jobs && jobs[j + 1].block_start <= block) ++j;
        job = jobs[j];
        block -= job.block_start;
    }
    int tx, ty;
    tile_of_block(block, job.tiles_t, job.tiles_dm, remap, tx, ty);
    const int tid = threadIdx.x, wave = uniform(tid >> 6);
    const int i0 = ty * kRows;
    Tile k;
    k.lane = tid & 63;
    k.rows = min(kRows, job.n_dm - i0);
    k.n_chan = job.n_chan;
    k.delays = job.delays + (size_t)i0 * job.n_chan;
    k.rd = range_rsrc(k.delays, 4u * (uint32_t)k.rows * (uint32_t)job.n_chan);
    k.in = job.in;
    k.keep = job.keep;
    k.in_stride = job.in_stride;
    k.in_bytes = job.in_bytes;
    k.t0 = (int64_t)tx * T;
    k.omax = job.omax;
    k.T = T;
    k.cols = (int)(job.n_out - k.t0 < T ? job.n_out - k.t0 : T);
    const int base = (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_raw;
    k.ring = base + wave * kWaveLds;
    const int next = base + kMatWaves * kWaveLds;
    // rows of sums, T columns and as many spare ones between two rows (and
    // before the first) as an addition may be off to either side
    const int spare = matrix_spare(job.omax), all = spare + kRows * (T + spare);
    k.pitch = T + spare;
    k.acc = next + 16 + 4 * spare;

    for (int q = tid; q < all / 4; q += 64 * kMatWaves) *lds<lds_w4>(next + 16 + 16 * q) = v4i{0, 0, 0, 0};
    if (tid == 0) {
        *lds<lds_i>(next) = kMatWaves;
        *lds<lds_i>(next + kKept) = 0;
        *lds<lds_i>(next + kPasses) = 0;
        *lds<lds_i>(next + kAsidePasses) = 0;
    }
    if (tid < 8) *lds<lds_i>(base + kAside + 4 * tid) = 0;
    __syncthreads();

    k.count = k.n_chan;
    k.order = k.row0 = 0;
    tasks<NS, false>(k, base, next, job.mat_parts, wave);
    __syncthreads();
    if (*lds<lds_i>(next + kAsidePasses) != 0) {
        // (32-bit staging offsets from the window's first channel)
        const int window = min(kWindow, (int)(kMaxStageSpan / k.in_stride) / kGroup * kGroup);
        for (; k.row0 < k.n_chan; k.row0 += window) {
            regroup(k, base, next, window, NS);
            tasks<NS, true>(k, base, next, job.mat_parts, wave);
            __syncthreads();
        }
    }

    // From sums of kStartSum - 128 * (sample - 128), low and high words of
    // 64-bit numbers whose low words never reach 2^32, to sums of samples.
    const int bias = 128 * (k.keep ? *lds<lds_i>(next + kKept) : k.n_chan) + (kStartSum / 128) * *lds<lds_i>(next + kPasses);
    const auto sum = [&](uint32_t v) { return bias - (int)(v >> 7); };
    if (job.dd_stride % 4 == 0 && ((uintptr_t)job.dd & 15) == 0) {
        for (int q = tid; q < k.rows * (T / 4); q += 64 * kMatWaves) {
            const int row = q / (T / 4), t = 4 * (q - row * (T / 4));
            const v4i x = *lds<lds_v4>(k.acc + 4 * (row * k.pitch + t));
            const v4i v = {sum((uint32_t)x[0]), sum((uint32_t)x[1]), sum((uint32_t)x[2]), sum((uint32_t)x[3])};
            int32_t *out = job.dd + (size_t)(i0 + row) * job.dd_stride + k.t0 + t;
            if (t + 4 <= k.cols) {
                *reinterpret_cast<v4i *>(out) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (t + e < k.cols) out[e] = v[e];
            }
        }
    } else {
        for (int q = tid; q < k.rows * T; q += 64 * kMatWaves) {
            const int row = q / T, t = q - row * T;
            if (t < k.cols)
                job.dd[(size_t)(i0 + row) * job.dd_stride + k.t0 + t] = sum(*lds<lds_u>(k.acc + 4 * (row * k.pitch + t)));
        }
    }
}

}  // namespace

namespace {

struct Sizes {
    int64_t n_dm, n_out;
};

// Row length of problems that run in one launch.  A work-group fills a CU, so a
// launch takes rounds of 256; in each it takes the time of about T + omax / 2
// columns plus its delays', passes' and last step's, about 400 columns' more.
// The length with the least of both: rounds that are full, and otherwise the
// longest that the LDS holds.  (With T = 640 throughout, 1024 trials x 6104
// samples were 320 work-groups, and took 1280 columns' time where two rounds of
// 384 do.)  0: none fits.
int row_length(const Sizes *problems, size_t n, int omax)
{
    int64_t longest = 0, best = 0;
    for (size_t k = 0; k < n; ++k) longest = std::max(longest, problems[k].n_out);
    int T = 0;
    for (int t = 128; matrix_lds_bytes(t, omax) <= kMaxLdsBytes; t += 8) {
        int64_t blocks = 0;
        for (size_t k = 0; k < n; ++k)
            blocks += (problems[k].n_dm + kRows - 1) / kRows * ((problems[k].n_out + t - 1) / t);
        const int64_t cost = (blocks + 255) / 256 * (t + omax / 2 + 400);
        if (T == 0 || cost < best) {
            best = cost;
            T = t;
        }
        if (t >= longest) break;
    }
    return T;
}

}  // namespace

int xcd_remap_setting()
{
    const char *e = getenv("AMBER_XCD_REMAP");
    return e ? atoi(e) : 1;
}

// When the matrix cores do it: what the vector kernel takes does not depend on
// the remainders, what this one takes grows with them and has a part per
// work-group that few channels do not repay.  With `most` (the remainders at
// the band's narrow end) and 64 .. 2048 trials x 2048 or 8192 samples, vector
// kernel's time over this one's:
//
//   channels   most 3-5     7        9.5-12     17         22         32
//   1536       2.4-3.3   1.8-2.5    1.1-1.9
//    768       2.3-3.0   2.0-2.6    1.4-2.0               0.6-1.0
//    384                 2.0-2.4    1.6-2.1               0.8-1.1
//    256                            1.4-1.7   1.03-1.28              0.6-0.85
//    128                                      0.79-1.0               0.6-0.8
//
// so: 256 channels or more, and `most` up to 18.  (`most` is an estimate from
// the table's summary that only the speed depends on.)
//
// A group's columns are its tile's and omax / 2 more on average, which counts
// where large shifts leave the LDS short rows: the more the more rounds of 256
// work-groups there are, as each reads a window of its own.  With `most` times
// (1 + omax / 2 / longest row), steps of 2 pc/cm3, vector kernel's time over this
// one's for ascending / descending frequencies:
//
//   channels  weighted   41 x 2860, 64 x 8192   400 x 12000, 1000 x 3000   1024 x 12208
//   1536        40       1.7-1.8 / 1.04         1.45 / 1.3-1.4             0.92 / 0.92
//   1347        44       1.4-1.6 / 1.0          1.25 / 1.2                 0.79 / 0.77
//   1152        50       1.25-1.35 / 0.99       1.06 / 1.0                 0.67 / 0.65
//   1024        56       1.1-1.2 / 0.9          0.96 / 0.9                 0.60 / 0.58
//
// so: any up to two rounds, up to 51 to four, else up to 38 (33, 1024 channels:
// 1.0-1.25).
//
// The estimate holds for channels in order of frequency at 1250-1550 MHz.  Wide
// bands have more remainders at their bottom than it says, other orders before
// they are sorted.  Same sizes and 64 x 2048, vector kernel's time over this
// one's with `most` 3-4.5 / 6.5-9 / 12 / 17.9:
//
//   300-1200 MHz                      1.3-2.4  1.3-1.9  1.2-1.7  0.85-1.25
//   shuffled or sub-bands in turn
//     512 .. 1536 channels            1.4-2.6  1.2-2.4  0.6-1.8  0.8-1.0
//     256 channels                    0.7-1.5  0.9-1.4  0.85-1.2 0.7-0.95
//
// (without the sorting 0.05-0.16 from 6.5 on, 0.65-1.0 below)
void use_matrix(const amber_delay_info &info, int64_t in_stride, int64_t n_out, bool automatic, DedispPlan *p)
{
    if (p->in_u16 || p->direct || n_out < 1) return;
    if (!automatic && p->dpb * p->dpt != kRows) return;  // explicit tiles choose the trials per work-group
    const int64_t omax = (int64_t)(kRows - 1) * info.max_step;
    // 32-bit staging offsets, 16-bit remainders, 32-bit biased sums
    if (64 * in_stride > kMaxStageSpan || omax >= 16384 || info.n_chan > 8192) return;
    // the largest step of a trial: max_step is rounded up to a whole sample,
    // the whole table's slope is not
    double rate = info.max_step;
    if (info.n_dm > 1) rate = std::min(rate, (double)info.max_delay / (info.n_dm - 1));
    // 16 channels off the middle one, 31 trials; 1.37: the delay's slope at
    // 1250 .. 1550 MHz is that much above its mean at the narrow end
    const double most = 2.0 + 1.37 * rate * (kRows - 1) / info.n_chan * kGroup / 2;
    if (info.n_chan < 256 || most > 18) return;
    // the longest rows that the LDS holds
    const int64_t longest = (kMaxLdsBytes - matrix_lds_bytes(0, (int)omax)) / (4 * kRows);
    if (longest < 128) return;
    const int64_t blocks = (int64_t)((info.n_dm + kRows - 1) / kRows) * ((n_out + longest - 1) / longest);
    const double weighted = most * (1.0 + 0.5 * (double)omax / (double)longest);
    if (blocks > 512 && weighted > (blocks > 1024 ? 38.0 : 51.0)) return;
    // remainders per pass: more take registers (and reads) that a band with
    // fewer does not need; one pass of 12 takes less than two of 7
    const int mat = most < 5.1 ? 5 : most < 7.1 ? 7 : most < 9.1 ? 9 : 12;
    // explicit tiles of up to 256 samples choose that
    const Sizes size{info.n_dm, n_out};
    const int T = !automatic && p->tile_t <= 256 ? 256 : row_length(&size, 1, (int)omax);
    if (T == 0 || matrix_lds_bytes(T, (int)omax) > kMaxLdsBytes) return;
    p->mat = mat;
    p->omax = (int)omax;
    p->dpb = 16;
    p->dpt = 2;
    p->tile_t = T;
    p->lds_bytes = matrix_lds_bytes(T, (int)omax);
    // few groups: column ranges of each, so that every wavefront has two tasks
    const int groups = (info.n_chan + kGroup - 1) / kGroup;
    p->mat_parts = std::max(1, std::min(4, 2 * kMatWaves / groups));
}

// Beams of one launch set.  Those with the same explicit tiles stay one launch:
// all of them take the matrix cores, or none.  Those with automatic tiles run in
// one launch for each form of the kernel (remainders per pass).  With a row
// length and a launch for each beam, 8 beams of 512 channels x 256 trials x 3000
// to 7900 samples took 168 us where one launch takes 101, 16 of 256 x 64 x 2000
// to 7000 90 and 53.
void use_matrix_together(const std::vector<MatrixUse> &beams, std::vector<DedispPlan> *plans)
{
    const size_t n = beams.size();
    std::vector<DedispPlan> m = *plans;
    for (size_t k = 0; k < n; ++k)
        use_matrix(*beams[k].info, beams[k].in_stride, beams[k].n_out, beams[k].tiles == nullptr, &m[k]);
    const auto same = [&](size_t a, size_t b) {
        const amber_tiles *x = beams[a].tiles, *y = beams[b].tiles;
        if (!x || !y) return !x && !y && m[a].mat == m[b].mat;
        return x->threads_per_dm == y->threads_per_dm && x->samples_per_thread == y->samples_per_thread &&
               x->dms_per_block == y->dms_per_block && x->channel_unroll == y->channel_unroll &&
               x->dms_per_thread == y->dms_per_thread && x->direct_reads == y->direct_reads;
    };
    std::vector<char> done(n, 0);
    for (size_t k = 0; k < n; ++k) {
        if (done[k]) continue;
        bool all = true;
        int mat = 0, omax = 0;
        std::vector<size_t> set;
        std::vector<Sizes> sizes;
        for (size_t j = k; j < n; ++j) {
            if (done[j] || !same(k, j)) continue;
            done[j] = 1;
            set.push_back(j);
            sizes.push_back({beams[j].info->n_dm, beams[j].n_out});
            all = all && m[j].mat != 0;
            mat = std::max(mat, m[j].mat);
            omax = std::max(omax, m[j].omax);
        }
        if (!all) continue;
        const bool short_rows = beams[k].tiles && (*plans)[k].tile_t <= 256;
        const int T = set.size() == 1 ? m[k].tile_t : short_rows ? 256 : row_length(sizes.data(), sizes.size(), omax);
        for (size_t j : set) {
            (*plans)[j] = m[j];
            (*plans)[j].mat = mat;
            (*plans)[j].tile_t = T;
            (*plans)[j].lds_bytes = matrix_lds_bytes(T, m[j].omax);
        }
    }
}

amber_status launch_dedisperse_matrix_jobs(const DedispPlan &p, const DedispJob *single, const DedispJob *d_jobs,
                                           int n_jobs, int64_t n_blocks, int64_t lds_bytes, hipStream_t stream)
{
    if (n_blocks > 0x7fffffff) return fail(AMBER_E_SHAPE, "grid of %lld work-groups is too large", (long long)n_blocks);
    const int lds = (int)lds_bytes;
    const auto kernel = p.mat <= 5   ? dedisperse_matrix_kernel<5>
                        : p.mat <= 7 ? dedisperse_matrix_kernel<7>
                        : p.mat <= 9 ? dedisperse_matrix_kernel<9>
                                     : dedisperse_matrix_kernel<12>;
    AMBER_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  lds),
              "hipFuncSetAttribute(dedisperse_matrix)");
    static const int remap = xcd_remap_setting();
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_blocks), dim3(64 * kMatWaves), (size_t)lds, stream,
                       single ? *single : DedispJob{}, d_jobs, n_jobs, p.tile_t, d_jobs ? 0 : remap);
    AMBER_HIP(hipGetLastError(), "dedisperse (matrix) launch");
    return AMBER_OK;
}

}  // namespace amber
