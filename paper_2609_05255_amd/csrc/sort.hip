// Depth-sorted per-tile lists (Sec. 3.1 "depth-sorted order"): the pairs must
// come out ordered by (tile, depth key, Gaussian index).
//
// Instead of radix-sorting P 45-bit (tile, depth) keys, the Gaussians are
// sorted once by depth (4 stable 8-bit LSD passes over n 32-bit keys with the
// index, and beside it the tile rectangle, as value, so equal depths stay in index
// order). Then, in that order,
// each Gaussian gets one entry per 4x4-tile block its rectangle meets (about a
// quarter as many entries as pairs), a stable LSD sort on the block id groups
// the entries by block with depth order kept inside each block, and every
// block's 16 tile lists are cut out of its entries by ordered (ballot)
// compaction, each list written once, at its final place.
//
// One radix pass = k_radix_hist (per-workgroup digit counts and their sums over
// groups of workgroups) + k_radix_scatter: each workgroup adds up the counts
// before its own, each wave ranks a contiguous slice of the workgroup's keys
// with ballot-matched digits (no workgroup barrier per round), the workgroup
// reorders its 4096 to 16384 keys by digit in LDS, and writes each digit's run to
// consecutive global addresses. The grids are sized for the most keys a call can
// meet (the capacity, for the block entries); workgroups past the device-side
// count do nothing, and their rows are not read. A single-pass block sort's
// scatter has one workgroup more, which writes the tile lists' segment table
// from that pass's digit totals (the blocks' entry counts).
//
// With few Gaussians one workgroup sorts them by depth in LDS, and each block
// finds its own entries among all of them (k_small_depth_sort, k_small_counts, k_small_lists).
#include "gs_internal.h"

namespace gsr {

namespace {

constexpr int kDupItems = kDupChunk / kBlock;              // 4 per thread

__device__ __forceinline__ uint64_t lanemask_lt() { return (1ull << __lane_id()) - 1ull; }

// Exclusive scan of one u32 per thread over the 256-thread workgroup.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds4, uint32_t* total)
{
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds4[wave] = x;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t s = lds4[w];
        if (w < wave) before += s;
        tot += s;
    }
    __syncthreads();
    if (total) *total = tot;
    return before + x - v;
}

constexpr int kListThreads = 1024;   // radix passes, single-workgroup scans

// Exclusive scan of one value per thread over a 1024-thread workgroup.
template <typename T>
__device__ __forceinline__ T wg_excl_scan_1024(T v, T* lds16, T* total)
{
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds16[wave] = x;
    __syncthreads();
    T before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kListThreads / kWave; ++w) {
        const T s = lds16[w];
        if (w < wave) before += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return before + x - v;
}

// Lanes of this wave holding the same kBits-bit digit (restricted to valid lanes).
template <int kBits>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid)
{
    const uint64_t v = __ballot(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < kBits; ++b) {
        const uint32_t bit = (d >> b) & 1u;
        const uint64_t bm = __ballot(bit);
        const uint32_t s = 0u - bit;   // all ones where this lane's bit is set
        // keep the lanes whose bit equals ours: bm where set, ~bm where clear
        lo &= ~((uint32_t)bm ^ s);
        hi &= ~((uint32_t)(bm >> 32) ^ s);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Digit counts of each workgroup's keys, one row of R counts per workgroup, and
// their sums over groups of `group` workgroups (sup, zeroed beforehand), from
// which the scatter takes its digits' positions: about sqrt(workgroups) rows of
// either kind. A kernel of its own that scanned each digit's counts over the
// workgroups took 5 us and a launch per pass at any size; adding the rows up in
// the scatter costs about 1 us of it.
template <int kBits, int kItems>
__global__ __launch_bounds__(kListThreads) void k_radix_hist(const uint32_t* __restrict__ keys, PairCount cnt, int shift,
                                                       uint32_t* __restrict__ hist, uint32_t* __restrict__ sup,
                                                       int group)
{
    constexpr int R = 1 << kBits;
    constexpr int kTile = kListThreads * kItems;
    const uint64_t count = cnt.get();
    if ((uint64_t)blockIdx.x * kTile >= count) return;   // past the keys: the scatter does not read it
    // 16 copies of the counts (per wave % 4 and lane % 4): a skewed digit, such
    // as the exponent byte of the depth keys, then meets at most 16 lanes of an
    // instruction on one counter
    __shared__ uint32_t h[16][R];
    for (int k = threadIdx.x; k < 16 * R; k += kListThreads) (&h[0][0])[k] = 0;
    __syncthreads();
    const int copy = ((threadIdx.x >> 6) & 3) * 4 + (threadIdx.x & 3);
    const uint64_t base = (uint64_t)blockIdx.x * kTile;
    // all loads first (one memory round trip), then the counts
    uint32_t k[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint64_t idx = base + (uint64_t)r * kListThreads + threadIdx.x;
        k[r] = idx < count ? keys[idx] : 0u;
    }
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint64_t idx = base + (uint64_t)r * kListThreads + threadIdx.x;
        if (idx < count) atomicAdd(&h[copy][(k[r] >> shift) & (R - 1)], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < R; d += kListThreads) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) c += h[w][d];
        hist[(size_t)blockIdx.x * R + d] = c;
        if (c) atomicAdd(&sup[(size_t)(blockIdx.x / (unsigned)group) * R + d], c);
    }
}

// Column sums of every step-th row from r0 below r1 of a table of R-wide rows,
// by one wave, into out[R]: its lanes take 16 bytes of a row each, several rows
// in flight together.
template <int R>
__device__ __forceinline__ void sum_rows(const uint32_t* __restrict__ rows, int r0, int r1, int step, uint32_t* out)
{
    constexpr int kVec = R >= 4 ? 4 : R;                      // columns per load
    constexpr int kCols = R / kVec;                           // loads per row
    constexpr int kPer = kCols > kWave ? kCols / kWave : 1;   // loads per lane and row
    constexpr int kFly = 4;                                   // rows in flight
    const int lane = __lane_id();
    if (lane >= kCols) return;
    uint32_t sum[kPer][kVec] = {};
    for (int r = r0; r < r1; r += step * kFly) {
        uint32_t v[kFly][kPer][kVec];
#pragma unroll
        for (int u = 0; u < kFly; ++u)
#pragma unroll
            for (int q = 0; q < kPer; ++q)
#pragma unroll
                for (int j = 0; j < kVec; ++j)
                    v[u][q][j] = r + u * step < r1 ? rows[(size_t)(r + u * step) * R + (q * kWave + lane) * kVec + j] : 0u;
#pragma unroll
        for (int u = 0; u < kFly; ++u)
#pragma unroll
            for (int q = 0; q < kPer; ++q)
#pragma unroll
                for (int j = 0; j < kVec; ++j) sum[q][j] += v[u][q][j];
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q)
#pragma unroll
        for (int j = 0; j < kVec; ++j) out[(q * kWave + lane) * kVec + j] = sum[q][j];
}

// The block entries' segment table (see k_segments), written by one extra
// workgroup of the block sort's scatter from that pass's digit totals.
struct SegTable {
    uint32_t* block_ranges;   // nullptr: no table
    uint32_t* seg_base;
    uint32_t* seg_block;
    uint32_t* counters;
    int n_blocks;
};

__device__ void segment_table(const uint32_t* block_count, const SegTable& t);

// A tile rectangle (x0 | y0 << 16, x1 | y1 << 16, half-open, not empty) of a
// grid of at most 256 x 256 tiles in 32 bits: x0, y0, x1 - 1, y1 - 1. The
// empty rectangle of a culled Gaussian has x0 above x1 - 1.
constexpr uint32_t kEmptyRect32 = 0x0000FFFFu;

__device__ __forceinline__ uint32_t pack_rect32(uint2 r)
{
    return (r.x & 0xFFu) | ((r.x >> 8) & 0xFF00u) | (((r.y & 0xFFFFu) - 1u) << 16) | (((r.y >> 16) - 1u) << 24);
}

__device__ __forceinline__ uint2 unpack_rect32(uint32_t p)
{
    if (p == kEmptyRect32) return make_uint2(0u, 0u);
    return make_uint2((p & 0xFFu) | ((p << 8) & 0xFF0000u), (((p >> 16) & 0xFFu) + 1u) | (((p >> 24) + 1u) << 16));
}

// The values a pass moves: the Gaussian's index alone, or with it its packed
// tile rectangle (x: index, y: rectangle).
__device__ __forceinline__ uint32_t value_index(uint32_t v) { return v; }
__device__ __forceinline__ uint32_t value_index(uint2 v) { return v.x; }

// What a scatter pass does beside moving keys and values.
enum PassMode {
    kPlain,
    kFirst,    // first depth pass: makes the values, (index, packed rectangle read from the record in index order)
    kGather,   // last depth pass of a grid beyond 256 tiles a side: gathers the rectangles into depth order
};

__device__ __forceinline__ uint2 splat_rect(const gs_splat* __restrict__ splats, uint32_t i)
{
    return *reinterpret_cast<const uint2*>(reinterpret_cast<const uint32_t*>(splats + i) + kSplatRectWord);
}

// keys_out == nullptr drops the keys; vals_in == nullptr means value = position.
template <int kBits, int kItems, typename ValT, int kMode>
__global__ __launch_bounds__(kListThreads) void k_radix_scatter(const uint32_t* __restrict__ keys_in,
                                                          const ValT* __restrict__ vals_in, PairCount cnt, int shift,
                                                          const uint32_t* __restrict__ hist,
                                                          const uint32_t* __restrict__ sup, int group,
                                                          uint32_t* __restrict__ keys_out, ValT* __restrict__ vals_out,
                                                          const gs_splat* __restrict__ splats,
                                                          uint2* __restrict__ rect_out, SegTable seg)
{
    constexpr int R = 1 << kBits;
    constexpr int kTile = kListThreads * kItems;
    constexpr int kWaves = kListThreads / kWave;
    constexpr int kSlice = kTile / kWaves;   // keys per wave
    __shared__ uint32_t wcnt[kWaves][R];      // per-wave digit counts, then each wave's first place of each digit
    __shared__ uint32_t gbase[R];        // global position of a digit's first key, less its place in the workgroup
    __shared__ ValT buf[kTile];          // row sums, then the workgroup's keys, then its values, in digit order
    __shared__ uint32_t lds16[kWaves];
    static_assert(sizeof(buf) >= kWaves * R * sizeof(uint32_t), "row sums");
    uint32_t (*part)[R] = reinterpret_cast<uint32_t (*)[R]>(buf);
    uint32_t* kbuf = reinterpret_cast<uint32_t*>(buf);
    const uint64_t count = cnt.get();
    const int t = threadIdx.x, wave = t >> 6, lane = __lane_id();
    // digits t * kDPT + j (consecutive per thread)
    constexpr int kDPT = R > kListThreads ? R / kListThreads : 1;
    const int d0 = t * kDPT;
    const int active = (int)min((uint64_t)0x7FFFFFFF, (count + kTile - 1) / kTile);
    const int nsup = (active + group - 1) / group;
    if (seg.block_ranges && blockIdx.x == gridDim.x - 1) {   // the extra workgroup
        sum_rows<R>(sup, wave, nsup, kWaves, part[wave]);
        __syncthreads();
        for (int d = t; d < R; d += kListThreads) {
            uint32_t c = 0;
            for (int w = 0; w < kWaves; ++w) c += part[w][d];
            gbase[d] = c;
        }
        __syncthreads();
        segment_table(gbase, seg);
        return;
    }
    if ((uint64_t)blockIdx.x * kTile >= count) return;   // past the keys: nothing to move
    // the keys' loads first: they are in flight while the counts are added up
    const uint64_t base = (uint64_t)blockIdx.x * kTile;
    const uint64_t wbase = base + (uint64_t)wave * kSlice;
    uint32_t key[kItems];
    ValT val[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint64_t idx = wbase + (uint64_t)i * kWave + lane;
        key[i] = idx < count ? keys_in[idx] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint64_t idx = min(wbase + (uint64_t)i * kWave + lane, count - 1);   // no condition: loads together
        if constexpr (kMode == kFirst) {
            const uint2 r = splat_rect(splats, (uint32_t)idx);
            val[i] = make_uint2(r.x, r.y);   // packed below
        } else if constexpr (sizeof(ValT) == 4) {
            val[i] = vals_in ? vals_in[idx] : (uint32_t)idx;
        } else {
            val[i] = vals_in[idx];
        }
    }
    // 4 waves add up the group sums before this workgroup's group, 4 the others,
    // 8 the counts of its group before it
    {
        const int sb = (int)blockIdx.x / group;
        if (wave < 4) sum_rows<R>(sup, wave, sb, 4, part[wave]);
        else if (wave < 8) sum_rows<R>(sup, sb + wave - 4, nsup, 4, part[wave]);
        else sum_rows<R>(hist, sb * group + wave - 8, (int)blockIdx.x, 8, part[wave]);
    }
    __syncthreads();
    uint32_t tot[kDPT] = {}, before[kDPT] = {}, dsum = 0;
#pragma unroll
    for (int j = 0; j < kDPT; ++j)
        if (d0 + j < R) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t b = part[w][d0 + j];
                before[j] += b + part[8 + w][d0 + j] + part[12 + w][d0 + j];
                tot[j] += b + part[4 + w][d0 + j];
            }
            dsum += tot[j];
        }
    uint32_t total;
    uint32_t dbase = wg_excl_scan_1024(dsum, lds16, &total);   // its barriers end the use of part
#pragma unroll
    for (int j = 0; j < kDPT; ++j) {
        const int d = d0 + j;
        if (d < R) {
            gbase[d] = dbase + before[j];
            for (int w = 0; w < kWaves; ++w) wcnt[w][d] = 0;
        }
        dbase += tot[j];
    }
    __syncthreads();
    // rank within the wave's slice, in key order
    uint32_t rank[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint64_t idx = wbase + (uint64_t)i * kWave + lane;
        const bool valid = idx < count;
        const uint32_t d = (key[i] >> shift) & (R - 1);
        const uint64_t peers = match_digit<kBits>(d, valid);
        const uint32_t r = (uint32_t)__popcll(peers & lanemask_lt());
        const uint32_t pre = valid ? wcnt[wave][d] : 0u;
        rank[i] = pre + r;
        if (valid && r == 0) wcnt[wave][d] = pre + (uint32_t)__popcll(peers);
        // the next round reads counts this round's leaders wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t tsum = 0;
#pragma unroll
    for (int j = 0; j < kDPT; ++j)
        if (d0 + j < R)
            for (int w = 0; w < kWaves; ++w) tsum += wcnt[w][d0 + j];
    uint32_t ls = wg_excl_scan_1024(tsum, lds16, &total);
#pragma unroll
    for (int j = 0; j < kDPT; ++j) {
        const int d = d0 + j;
        if (d < R) {
            gbase[d] -= ls;
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t c = wcnt[w][d];
                wcnt[w][d] = ls;
                ls += c;
            }
        }
    }
    __syncthreads();
    // place in the workgroup's digit order; then the keys and the values go
    // through one LDS buffer in turn (one each would halve the resident
    // workgroups), each digit's run to consecutive addresses
    const uint32_t nvalid = (uint32_t)min((uint64_t)kTile, count - base);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint64_t idx = wbase + (uint64_t)i * kWave + lane;
        if (idx < count) {
            rank[i] += wcnt[wave][(key[i] >> shift) & (R - 1)];
            kbuf[rank[i]] = key[i];
        }
    }
    __syncthreads();
    uint32_t pos[kItems], culled = 0;   // culled: bit i, the key of the i-th key written is ~0
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint32_t j = t + i * kListThreads;
        pos[i] = 0;
        if (j < nvalid) {
            const uint32_t k = kbuf[j];
            pos[i] = gbase[(k >> shift) & (R - 1)] + j;
            if (keys_out) keys_out[pos[i]] = k;
            if (kMode == kGather) culled |= (k == 0xFFFFFFFFu ? 1u : 0u) << i;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint64_t idx = wbase + (uint64_t)i * kWave + lane;
        if constexpr (kMode == kFirst)
            val[i] = make_uint2((uint32_t)idx, key[i] != 0xFFFFFFFFu ? pack_rect32(val[i]) : kEmptyRect32);
        if (idx < count) buf[rank[i]] = val[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint32_t j = t + i * kListThreads;
        if (j < nvalid) {
            const ValT v = buf[j];
            vals_out[pos[i]] = v;
            // culled Gaussians (key ~0, no splat record) get an empty rectangle
            if (kMode == kGather)
                rect_out[pos[i]] = (culled >> i) & 1u ? make_uint2(0u, 0u) : splat_rect(splats, value_index(v));
        }
    }
}

// One stable LSD pass over kBits bits at `shift`. The grids are sized for
// cnt.host keys (the capacity in device mode). `sup`: this pass's group sums,
// zeroed.
template <int kBits, int kItems, typename ValT, int kMode>
void radix_pass(const uint32_t* keys_in, const ValT* vals_in, PairCount cnt, int shift, uint32_t* keys_out,
                ValT* vals_out, uint32_t* hist, uint32_t* sup, hipStream_t s, const gs_splat* splats = nullptr,
                uint2* rect_out = nullptr, SegTable seg = SegTable{nullptr, nullptr, nullptr, nullptr, 0})
{
    static_assert(kItems <= 32, "one culled bit per key");
    const int nblocks = (int)std::max<int64_t>(div_up((int64_t)cnt.host, (int64_t)kListThreads * kItems), 1);
    const int group = radix_group(nblocks);
    hipLaunchKernelGGL((k_radix_hist<kBits, kItems>), dim3(nblocks), dim3(kListThreads), 0, s, keys_in, cnt, shift, hist, sup,
                       group);
    hipLaunchKernelGGL((k_radix_scatter<kBits, kItems, ValT, kMode>), dim3(nblocks + (seg.block_ranges ? 1 : 0)),
                       dim3(kListThreads), 0, s, keys_in, vals_in, cnt, shift, hist, sup, group, keys_out, vals_out, splats,
                       rect_out, seg);
}

// A block-sort pass over `bits` (1..9) bits.
constexpr int kBlockSortBits = 9;
template <int kItems>
static hipError_t block_radix_pass(const uint32_t* keys_in, const uint32_t* vals_in, PairCount cnt, int shift, int bits,
                                   uint32_t* keys_out, uint32_t* vals_out, uint32_t* hist, uint32_t* sup,
                                   hipStream_t s, SegTable seg)
{
    switch (bits) {
#define GS_PASS(b)                                                                                                \
    case b:                                                                                                       \
        radix_pass<b, kItems, uint32_t, kPlain>(keys_in, vals_in, cnt, shift, keys_out, vals_out, hist, sup, s,   \
                                                nullptr, nullptr, seg);                                           \
        break;
        GS_PASS(1) GS_PASS(2) GS_PASS(3) GS_PASS(4) GS_PASS(5) GS_PASS(6) GS_PASS(7) GS_PASS(8) GS_PASS(9)
#undef GS_PASS
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Keys per thread of the block sort: 8, or 16 where the capacity leaves room for
// millions of entries (about a quarter of the pairs), for longer runs per digit
// (scatter 12 us with 8 and 18 with 16 at 0.3M entries, 62 and 54 at 6.5M, 104
// and 82 at 11M). The number of entries is only known on the device: a buffer
// with room for many more pairs than there are gets 16 by its size (0.33M pairs:
// the whole binning 96 us with the capacity they need, 104 at 16M, 109 at 64M).
static int block_items(uint64_t capacity) { return capacity <= (12u << 20) ? kBlockSortItems : 2 * kBlockSortItems; }

// ---- block entries in depth order -------------------------------------------
//
// A block is kBlockDim x kBlockDim tiles. Each visible Gaussian gets one entry
// per block its tile rectangle meets, in depth order; the entries are then
// sorted by block id (stable, so depth order holds inside a block), and each
// block's tile lists are cut out of its entries by ordered compaction.

// Area of a packed rectangle (x0 | y0 << 16, x1 | y1 << 16, half-open).
__device__ __forceinline__ uint32_t rect_area(uint2 r)
{
    return ((r.y & 0xFFFFu) - (r.x & 0xFFFFu)) * ((r.y >> 16) - (r.x >> 16));
}

// Block rectangle (half-open, block units, packed like a tile rectangle) of a
// tile rectangle; an empty rectangle stays empty.
__device__ __forceinline__ uint2 block_rect(uint2 r)
{
    if (rect_area(r) == 0) return make_uint2(0u, 0u);
    const uint32_t x0 = r.x & 0xFFFFu, y0 = r.x >> 16, x1 = r.y & 0xFFFFu, y1 = r.y >> 16;
    constexpr uint32_t kS = 2, kR = kBlockDim - 1;   // log2 and mask of the block size
    static_assert(kBlockDim == 1 << kS, "block size");
    return make_uint2((x0 >> kS) | ((y0 >> kS) << 16), ((x1 + kR) >> kS) | (((y1 + kR) >> kS) << 16));
}

// Index and tile rectangle of the i-th Gaussian in depth order.
template <bool kPacked>
__device__ __forceinline__ uint2 sorted_rect_at(const DepthOrder& o, int64_t i)
{
    return kPacked ? unpack_rect32(o.packed[i].y) : o.rect[i];
}

// Entries of each chunk of kDupChunk depth-ordered Gaussians.
template <bool kPacked>
__global__ __launch_bounds__(kBlock) void k_entry_partial(DepthOrder order, int64_t n,
                                                          uint32_t* __restrict__ part)
{
    __shared__ uint32_t lds4[4];
    uint32_t sum = 0;
    for (int k = 0; k < kDupItems; ++k) {
        const int64_t i = (int64_t)blockIdx.x * kDupChunk + (int64_t)k * kBlock + threadIdx.x;
        if (i < n) sum += rect_area(block_rect(sorted_rect_at<kPacked>(order, i)));
    }
    uint32_t total;
    block_excl_scan(sum, lds4, &total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Exclusive scan of the per-chunk totals (one workgroup) of more than
// kSumChunks chunks; the grand total, the number of entries, goes to *entries (0
// when the pair count is over capacity: nothing downstream then reads an entry).
__global__ __launch_bounds__(kBlock) void k_scan_partials(uint32_t* __restrict__ part, int count, PairCount pairs,
                                                          uint64_t* __restrict__ entries)
{
    __shared__ uint32_t lds4[4];
    const int per = (count + kBlock - 1) / kBlock;
    const int start = threadIdx.x * per, end = min(start + per, count);
    uint32_t sum = 0;
    for (int k = start; k < end; ++k) sum += part[k];
    uint32_t total;
    uint32_t run = block_excl_scan(sum, lds4, &total);
    for (int k = start; k < end; ++k) {
        const uint32_t v = part[k];
        part[k] = run;
        run += v;
    }
    if (threadIdx.x == 0) *entries = pairs.overflow() ? 0ull : (uint64_t)total;
}

// Inclusive maximum scan over the wave's lanes (DPP row shifts, then the row
// broadcasts); lanes without a source keep their value.
__device__ __forceinline__ int wave_max_scan(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x111, 0xF, 0xF, false));   // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x112, 0xF, 0xF, false));   // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x114, 0xF, 0xF, false));   // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x118, 0xF, 0xF, false));   // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x142, 0xA, 0xF, false));   // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x143, 0xC, 0xF, false));   // row_bcast:31
    return v;
}

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bit 4k + i set where the tile rectangle r meets tile (4 bx + i, 4 by + k).
__device__ __forceinline__ uint32_t tile_mask(uint2 r, int bx, int by)
{
    const int ox = kBlockDim * bx, oy = kBlockDim * by;
    const int cx0 = max((int)(r.x & 0xFFFFu) - ox, 0), cx1 = min((int)(r.y & 0xFFFFu) - ox, kBlockDim);
    const int cy0 = max((int)(r.x >> 16) - oy, 0), cy1 = min((int)(r.y >> 16) - oy, kBlockDim);
    if (cx1 <= cx0 || cy1 <= cy0) return 0u;
    const uint32_t cols = ((1u << cx1) - 1u) & ~((1u << cx0) - 1u);
    const uint32_t rows = ((1u << cy1) - 1u) & ~((1u << cy0) - 1u);
    // rows bit k -> bit 4k, then one copy of the column bits per row
    const uint32_t spread = (rows & 1u) | ((rows & 2u) << 3) | ((rows & 4u) << 6) | ((rows & 8u) << 9);
    return cols * spread;
}

// Emits the entries of a chunk of depth-ordered Gaussians, each Gaussian's
// blocks in row-major order of its block rectangle: key = block id << 16 |
// the mask of the block's tiles that the Gaussian's rectangle meets, value =
// the Gaussian's index. The chunk's offsets, rectangles and indices are staged
// in LDS. Each wave then emits a contiguous quarter of the chunk's entries,
// kDupWin consecutive entries per round in groups of 64 (consecutive lanes
// write consecutive addresses): the lanes mark in LDS where the Gaussians of
// the next kDupWin - 1 slots start inside the round's window (after its first
// entry, which belongs to the round's first Gaussian), and an inclusive
// maximum scan over the window gives each entry its Gaussian. Depth order puts
// every culled Gaussian (no tiles) after the visible ones, so starts inside a
// window are distinct.
constexpr int kDupGroups = 8;                   // 64-entry groups per round
constexpr int kDupWin = kWave * kDupGroups;     // entries per round
constexpr int kMaskBits = 16;                   // low key bits: the tile mask

//
// Up to kSumChunks chunks each workgroup adds up the totals of the chunks before
// its own (kSum; a few loads per thread, against 5 us and a launch for a scan of
// them), and the last one stores the number of entries; a larger scene's totals
// are scanned beforehand, since the sums grow with the square of the chunks.
constexpr int kSumChunks = 8192;

template <bool kPacked, bool kSum>
__global__ __launch_bounds__(kBlock) void k_block_entries(DepthOrder order, int64_t n,
                                                          const uint32_t* __restrict__ part, int blocks_x,
                                                          PairCount pairs, uint64_t capacity,
                                                          uint64_t* __restrict__ entries, uint32_t* __restrict__ keys,
                                                          uint32_t* __restrict__ vals)
{
    // nothing is written when the pairs are over capacity
    const uint32_t count = pairs.overflow() ? 0u : (uint32_t)capacity;
    __shared__ uint32_t soff[kDupChunk + 1];
    __shared__ uint32_t sorg[kDupChunk];   // block rectangle origin x0 | y0 << 16
    __shared__ uint32_t swid[kDupChunk];   // block rectangle width
    __shared__ uint2 srect[kDupChunk];     // tile rectangle
    __shared__ uint32_t sgid[kDupChunk];   // Gaussian index
    __shared__ int smark[kBlock / kWave][kDupWin];
    __shared__ uint32_t lds4[4];
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kDupChunk;
    uint32_t cnt[kDupItems];
    uint32_t sum = 0;
    for (int k = 0; k < kDupItems; ++k) {
        const int slot = t * kDupItems + k;
        const int64_t i = base + slot;
        uint32_t c = 0, org = 0, w = 1, g = 0;
        uint2 tr = make_uint2(0u, 0u);
        if (i < n) {
            if (kPacked) {
                const uint2 v = order.packed[i];
                g = v.x;
                tr = unpack_rect32(v.y);
            } else {
                g = order.gid[i];
                tr = order.rect[i];
            }
            const uint2 r = block_rect(tr);
            c = rect_area(r);
            if (c != 0) {
                org = r.x;
                w = (r.y & 0xFFFFu) - (r.x & 0xFFFFu);
            }
        }
        cnt[k] = c;
        sum += c;
        sorg[slot] = org;
        swid[slot] = w;
        srect[slot] = tr;
        sgid[slot] = g;
    }
    uint32_t total;
    uint32_t off = block_excl_scan(sum, lds4, &total);
    for (int k = 0; k < kDupItems; ++k) {
        soff[t * kDupItems + k] = off;
        off += cnt[k];
    }
    if (t == 0) soff[kDupChunk] = total;
    __syncthreads();
    uint32_t gbase = 0;
    if (kSum) {
        uint32_t before = 0;
        for (uint32_t k = t; k < blockIdx.x; k += kBlock) before += part[k];
        block_excl_scan(before, lds4, &gbase);
        if (blockIdx.x == gridDim.x - 1 && t == 0) *entries = pairs.overflow() ? 0ull : (uint64_t)gbase + total;
    } else {
        gbase = part[blockIdx.x];
    }
    const int wave = t >> 6, lane = __lane_id();
    const uint32_t q0 = (uint32_t)(((uint64_t)total * wave) / (kBlock / kWave));
    const uint32_t q1 = (uint32_t)(((uint64_t)total * (wave + 1)) / (kBlock / kWave));
    if (q0 >= q1) return;
    // last slot whose offset is <= q0 (the same address in every lane)
    int lo = 0, hi = kDupChunk;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (soff[mid] <= q0) lo = mid;
        else hi = mid;
    }
    int first = lo;
    int* mark = smark[wave];
    for (uint32_t p0 = q0; p0 < q1; p0 += kDupWin) {
#pragma unroll
        for (int k = 0; k < kDupGroups; ++k) mark[kWave * k + lane] = (k == 0 && lane == 0) ? 0 : -1;
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < kDupGroups; ++k) {
            const int d = kWave * k + lane;   // slot offset from the round's first Gaussian
            const int sl = first + d;
            if (d > 0 && sl < kDupChunk) {
                const uint32_t o = soff[sl];
                if (o > p0 && o < p0 + kDupWin && soff[sl + 1] > o) mark[o - p0] = d;
            }
        }
        wave_lds_fence();
        // in stages, so each stage's LDS latency is paid once per round
        int m[kDupGroups];
#pragma unroll
        for (int k = 0; k < kDupGroups; ++k) m[k] = mark[kWave * k + lane];
        int run = 0;   // owner of the window's positions so far (mark[0] = 0)
#pragma unroll
        for (int k = 0; k < kDupGroups; ++k) {
            m[k] = max(wave_max_scan(m[k]), run);
            run = __builtin_amdgcn_readlane(m[k], kWave - 1);
        }
        uint32_t o[kDupGroups], w[kDupGroups], org[kDupGroups], gid[kDupGroups];
        uint2 tr[kDupGroups];
#pragma unroll
        for (int k = 0; k < kDupGroups; ++k) {
            const int slot = first + m[k];
            o[k] = soff[slot];
            w[k] = swid[slot];
            org[k] = sorg[slot];
            tr[k] = srect[slot];
            gid[k] = sgid[slot];
        }
#pragma unroll
        for (int k = 0; k < kDupGroups; ++k) {
            const uint32_t p = p0 + kWave * k + lane;
            const uint32_t i = p - o[k];
            // i / w by a float reciprocal, corrected to the exact quotient (an
            // entry index and a block-rectangle width are both below 2^16, so
            // the estimate is off by at most one)
            uint32_t q = (uint32_t)((float)i * __builtin_amdgcn_rcpf((float)w[k]));
            q = q * w[k] > i ? q - 1u : q;
            q = (q + 1u) * w[k] <= i ? q + 1u : q;
            const uint32_t bx = (org[k] & 0xFFFFu) + (i - q * w[k]);
            const uint32_t by = (org[k] >> 16) + q;
            const uint32_t out = gbase + p;
            if (p < q1 && out < count) {
                keys[out] = ((by * (uint32_t)blocks_x + bx) << kMaskBits) | tile_mask(tr[k], (int)bx, (int)by);
                vals[out] = gid[k];
            }
        }
        // the next round starts with the Gaussian holding entry p0 + kDupWin: the
        // window's last owner, or the one after it if that ends exactly there
        const int last = first + run;
        first = last + (soff[last + 1] == p0 + kDupWin ? 1 : 0);
        wave_lds_fence();   // this round's mark reads before the next round's clear
    }
}

// One wave per boundary v = 0..n_keys of sorted keys: the first position whose
// key >> shift is >= v, by a 64-way search. Each round the lanes probe 64 evenly spaced
// positions of [lo, hi); the probes below v form a prefix (the keys are
// sorted), so their count c narrows the answer to (probe c-1, probe c]. About
// log64(count) dependent loads instead of log2(count). Boundary v ends range
// v - 1 and starts range v.
__global__ __launch_bounds__(kBlock) void k_ranges(const uint32_t* __restrict__ sorted_keys, int shift,
                                                   PairCount cnt, int n_keys, uint32_t* __restrict__ ranges)
{
    const uint32_t count = (uint32_t)cnt.get();
    const int v = (int)blockIdx.x * (kBlock / kWave) + (int)(threadIdx.x >> 6);
    if (v > n_keys) return;
    const uint32_t lane = __lane_id();
    uint32_t lo = 0, hi = count;   // the answer lies in [lo, hi]
    while (hi > lo) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint32_t p = lo + lane * step;
        const bool below = p < hi && (sorted_keys[p] >> shift) < (uint32_t)v;
        const uint32_t c = (uint32_t)__popcll(__ballot(below));
        const uint32_t nlo = c ? lo + (c - 1) * step + 1 : lo;
        hi = min(hi, lo + c * step);
        lo = nlo;
    }
    if (lane == 0) {
        if (v < n_keys) ranges[2 * v] = lo;
        if (v > 0) ranges[2 * v - 1] = lo;
    }
}

// ---- tile lists out of the block entries ------------------------------------
//
// Each block's entries are cut into segments of kSegEntries, one workgroup
// per segment and one sub-segment of 512 entries per wave. k_tile_count
// counts, per sub-segment, the entries that meet each of the block's 16 tiles;
// k_tile_scan turns the counts into each sub-segment's offset inside each
// tile's list and each tile's length; k_tile_starts places the lists in tile
// order (the ranges); k_tile_emit writes every tile's Gaussians, in entry
// order, by ballot compaction.

constexpr int kBlockTiles = kBlockDim * kBlockDim;             // 16
constexpr int kSegRounds = 8;                                  // 64-entry rounds per wave
constexpr int kSegEntries = kSegRounds * kBlock;               // 2048 entries per segment
constexpr int kSubSegs = kBlock / kWave;                       // one sub-segment per wave
static_assert(kBlockTiles == 16, "tile masks are 16 bits");

// Segment table: one workgroup of kListThreads. seg_base[b] = first segment of
// block b (and seg_base[n_blocks] = their number), seg_block[s] = the block of
// segment s, counters[0] = the number of segments. block_count (a single-pass
// block sort's digit totals, which give the ranges too) or nullptr: the ranges
// are there.
__device__ void segment_table(const uint32_t* block_count, const SegTable& t)
{
    __shared__ uint32_t lds16s[kListThreads / kWave];
    uint32_t carry = 0, ecarry = 0;
    for (int b0 = 0; b0 < t.n_blocks; b0 += kListThreads) {
        const int b = b0 + (int)threadIdx.x;
        uint32_t len = 0;
        if (block_count) {
            len = b < t.n_blocks ? block_count[b] : 0u;
            uint32_t etotal;
            const uint32_t start = ecarry + wg_excl_scan_1024(len, lds16s, &etotal);
            if (b < t.n_blocks) {
                t.block_ranges[2 * b] = start;
                t.block_ranges[2 * b + 1] = start + len;
            }
            ecarry += etotal;
        } else if (b < t.n_blocks) {
            len = t.block_ranges[2 * b + 1] - t.block_ranges[2 * b];
        }
        const uint32_t ns = (len + kSegEntries - 1) / kSegEntries;
        uint32_t total;
        const uint32_t first = carry + wg_excl_scan_1024(ns, lds16s, &total);
        if (b < t.n_blocks) {
            t.seg_base[b] = first;
            for (uint32_t k = 0; k < ns; ++k) t.seg_block[first + k] = (uint32_t)b;
        }
        carry += total;
    }
    if (threadIdx.x == 0) {
        t.seg_base[t.n_blocks] = carry;
        t.counters[0] = carry;
    }
}

__global__ __launch_bounds__(kListThreads) void k_segments(SegTable t) { segment_table(nullptr, t); }

// The entry range of segment s: block b, entries [e0, e1).
struct Segment {
    uint32_t b, e0, e1;
};

__device__ __forceinline__ Segment segment_of(uint32_t s, const uint32_t* __restrict__ seg_block,
                                              const uint32_t* __restrict__ seg_base,
                                              const uint32_t* __restrict__ block_ranges)
{
    Segment g;
    g.b = seg_block[s];
    const uint32_t j = s - seg_base[g.b];
    const uint32_t end = block_ranges[2 * g.b + 1];
    g.e0 = block_ranges[2 * g.b] + j * (uint32_t)kSegEntries;
    g.e1 = min(g.e0 + (uint32_t)kSegEntries, end);
    return g;
}

// The tile masks (and, for the emission, the Gaussian indices) of this wave's
// kSegRounds x 64 entries of the segment; lanes past the segment get mask 0.
// All loads are issued together, at indices clamped into the segment.
template <bool kIds>
__device__ __forceinline__ void load_segment(const Segment& g, const uint32_t* __restrict__ ent_key,
                                             const uint32_t* __restrict__ ent_gid, uint32_t mask[kSegRounds],
                                             uint32_t gid[kSegRounds])
{
    const uint32_t w0 = g.e0 + (threadIdx.x >> 6) * (kSegRounds * kWave) + __lane_id();
    const uint32_t last = g.e1 - 1u;   // segments are never empty
#pragma unroll
    for (int r = 0; r < kSegRounds; ++r) {
        const uint32_t e = min(w0 + r * kWave, last);
        mask[r] = ent_key[e];
        if (kIds) gid[r] = ent_gid[e];
    }
#pragma unroll
    for (int r = 0; r < kSegRounds; ++r)
        mask[r] = w0 + r * kWave <= last ? mask[r] & ((1u << kMaskBits) - 1u) : 0u;
}

// k_tile_count: per wave (a sub-segment of kSegRounds x 64 entries), the
// entries meeting each tile of the block; lane l (< 16) writes the count of
// tile l to wave_cnt[(4 s + wave) * 16 + l]. Tile-major, so that a single count
// is live at a time.
__global__ __launch_bounds__(kBlock) void k_tile_count(const uint32_t* __restrict__ ent_key,
                                                       const uint32_t* __restrict__ block_ranges,
                                                       const uint32_t* __restrict__ seg_base,
                                                       const uint32_t* __restrict__ seg_block,
                                                       const uint32_t* __restrict__ counters,
                                                       uint32_t* __restrict__ wave_cnt)
{
    const uint32_t s = blockIdx.x;
    if (s >= counters[0]) return;
    const Segment g = segment_of(s, seg_block, seg_base, block_ranges);
    uint32_t mask[kSegRounds], gid[kSegRounds];
    load_segment<false>(g, ent_key, nullptr, mask, gid);
    const int lane = __lane_id();
    uint32_t mine = 0;
#pragma unroll
    for (int l = 0; l < kBlockTiles; ++l) {
        uint32_t c = 0;
#pragma unroll
        for (int r = 0; r < kSegRounds; ++r) c += (uint32_t)__popcll(__ballot((mask[r] >> l) & 1u));
        // c is uniform: take it as such before the per-lane select
        mine = lane == l ? (uint32_t)__builtin_amdgcn_readfirstlane(c) : mine;
    }
    if (lane < kBlockTiles) wave_cnt[((size_t)s * kSubSegs + (threadIdx.x >> 6)) * kBlockTiles + lane] = mine;
}

// One wave per block: lane 16 q + l holds tile l of the q-th quarter of the
// block's sub-segments (4 per segment, in entry order): it sums its quarter's
// counts (loads issued together), the quarters are scanned across q, and a
// second sweep turns wave_cnt into each sub-segment's exclusive offset inside
// the tile's list. The tile's length goes to tile_ranges[2 t + 1].
__global__ __launch_bounds__(kWave) void k_tile_scan(const uint32_t* __restrict__ seg_base, int n_blocks,
                                                     int blocks_x, int tiles_x, int tiles_y,
                                                     uint32_t* __restrict__ wave_cnt, uint32_t* __restrict__ tile_ranges)
{
    const int b = blockIdx.x;
    if (b >= n_blocks) return;
    const int lane = __lane_id(), q = lane >> 4, l = lane & 15;
    const uint32_t s0 = seg_base[b] * kSubSegs, s1 = seg_base[b + 1] * kSubSegs;
    const uint32_t per = (s1 - s0 + 3) / 4;
    const uint32_t a0 = min(s0 + per * q, s1), a1 = min(a0 + per, s1);
    uint32_t sum = 0;
    for (uint32_t sb = a0; sb < a1; sb += 8) {
        uint32_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = sb + k < a1 ? wave_cnt[(size_t)(sb + k) * kBlockTiles + l] : 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += v[k];
    }
    // exclusive scan of the quarter sums across q (lanes l, l + 16, l + 32, l + 48)
    uint32_t x = sum;
    uint32_t y = __shfl_up(x, 16);
    if (q >= 1) x += y;
    y = __shfl_up(x, 32);
    if (q >= 2) x += y;
    const uint32_t total = __shfl(x, 48 + l);
    uint32_t run = x - sum;
    for (uint32_t sb = a0; sb < a1; sb += 8) {
        uint32_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = sb + k < a1 ? wave_cnt[(size_t)(sb + k) * kBlockTiles + l] : 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (sb + k < a1) wave_cnt[(size_t)(sb + k) * kBlockTiles + l] = run;
            run += v[k];
        }
    }
    const int tx = kBlockDim * (b % blocks_x) + (l & 3), ty = kBlockDim * (b / blocks_x) + (l >> 2);
    if (q == 0 && tx < tiles_x && ty < tiles_y) tile_ranges[2 * ((int64_t)ty * tiles_x + tx) + 1] = total;
}

// One workgroup: exclusive scan of the tile lengths in tile order, written as
// [start, end) ranges. Each thread takes kStartsPer consecutive tiles per
// sweep (one sweep covers 8,192 tiles: every image up to 1448 x 1448 tiles of
// 16 pixels in one). Pairs over capacity (the preprocess's count, or the
// lengths' sum) leave every range empty and raise counters[1], which stops the
// emission.
constexpr int kStartsPer = 8;

__global__ __launch_bounds__(kListThreads) void k_tile_starts(int n_tiles, PairCount pairs, uint64_t capacity,
                                                              uint32_t* __restrict__ tile_ranges,
                                                              uint32_t* __restrict__ counters)
{
    __shared__ uint64_t lds16[kListThreads / kWave];
    __shared__ int over;
    if (threadIdx.x == 0) over = pairs.overflow() ? 1 : 0;
    uint64_t carry = 0;   // 64-bit sums: a sum past the capacity is detected, never wrapped
    for (int t0 = 0; t0 < n_tiles; t0 += kListThreads * kStartsPer) {
        const int tb = t0 + (int)threadIdx.x * kStartsPer;
        uint32_t len[kStartsPer];
        uint64_t sum = 0;
#pragma unroll
        for (int k = 0; k < kStartsPer; ++k) {
            len[k] = tb + k < n_tiles ? tile_ranges[2 * (tb + k) + 1] : 0u;
            sum += len[k];
        }
        uint64_t total;
        const uint64_t before = wg_excl_scan_1024(sum, lds16, &total);   // also orders `over`
        uint64_t start = carry + before;
#pragma unroll
        for (int k = 0; k < kStartsPer; ++k) {
            if (tb + k < n_tiles) {
                if (start + len[k] > capacity) over = 1;
                tile_ranges[2 * (tb + k)] = (uint32_t)start;
                tile_ranges[2 * (tb + k) + 1] = (uint32_t)(start + len[k]);
            }
            start += len[k];
        }
        carry += total;
    }
    __syncthreads();
    if (over) {
        for (int t = threadIdx.x; t < n_tiles; t += kListThreads) tile_ranges[2 * t] = tile_ranges[2 * t + 1] = 0u;
    }
    if (threadIdx.x == 0) counters[1] = over ? 1u : 0u;
}

template <bool kTileIds>
__global__ __launch_bounds__(kBlock) void k_tile_emit(const uint32_t* __restrict__ ent_key,
                                                      const uint32_t* __restrict__ ent_gid,
                                                      const uint32_t* __restrict__ block_ranges,
                                                      const uint32_t* __restrict__ seg_base,
                                                      const uint32_t* __restrict__ seg_block,
                                                      const uint32_t* __restrict__ counters, int blocks_x, int tiles_x,
                                                      const uint32_t* __restrict__ wave_off,
                                                      const uint32_t* __restrict__ tile_ranges,
                                                      uint32_t* __restrict__ values, uint32_t* __restrict__ tile_ids)
{
    const uint32_t s = blockIdx.x;
    if (s >= counters[0] || counters[1] != 0u) return;
    const Segment g = segment_of(s, seg_block, seg_base, block_ranges);
    const int bx = (int)(g.b % (uint32_t)blocks_x), by = (int)(g.b / (uint32_t)blocks_x);
    const int lane = __lane_id();
    // lane l: this wave's offset inside the list of tile l
    const uint32_t base_l =
        lane < kBlockTiles ? wave_off[((size_t)s * kSubSegs + (threadIdx.x >> 6)) * kBlockTiles + lane] : 0u;
    uint32_t mask[kSegRounds], gid[kSegRounds];
    load_segment<true>(g, ent_key, ent_gid, mask, gid);
    const uint64_t below = (1ull << lane) - 1ull;
    // tile-major: one running offset live at a time
#pragma unroll
    for (int l = 0; l < kBlockTiles; ++l) {
        const uint32_t tile = (uint32_t)((kBlockDim * by + (l >> 2)) * tiles_x + kBlockDim * bx + (l & 3));
        uint32_t m_any = 0;
#pragma unroll
        for (int r = 0; r < kSegRounds; ++r) m_any |= (mask[r] >> l) & 1u;
        if (__ballot(m_any) == 0) continue;
        // the tile is inside the grid: some entry meets it
        uint32_t off = tile_ranges[2 * tile] + __builtin_amdgcn_readlane(base_l, l);
#pragma unroll
        for (int r = 0; r < kSegRounds; ++r) {
            const bool on = (mask[r] >> l) & 1u;
            const uint64_t m = __ballot(on);
            // inside the tile's range: the counts are those k_tile_count took,
            // and k_tile_starts let no range past the capacity
            if (on) {
                const uint32_t pos = off + (uint32_t)__popcll(m & below);
                values[pos] = gid[r];
                if (kTileIds) tile_ids[pos] = tile;
            }
            off += (uint32_t)__popcll(m);
        }
    }
}

// ---- few Gaussians ------------------------------------------------------------
//
// With few Gaussians the path above is bound by its 17 launches (4 to 5 us each).
// Up to kSmallSort one workgroup sorts the Gaussians by depth in LDS instead (11
// us at 1,024, 46 at 12,000; the passes above take 57 and 69 there, and overtake
// it where a workgroup's registers run out). Up to kSmallMax one workgroup per
// 4x4-tile block then finds the block's entries among all Gaussians, twice: to
// count its tile lists and to write them. Both are for grids whose rectangles are
// packed. The whole binning, this way / with the depth order and the block
// entries of the path above (us; lists of a few and of all Gaussians): 4,096
// Gaussians in 16 tiles 37 / 53, in 1,200 tiles 33 / 64 and 41 / 153; 12,288 in
// 16 tiles 82 to 84 / 80, in 1,200 tiles 67 / 90 and 94 / 191.
constexpr int kSmallSortItems = 12, kSmallItems = 24;             // keys per thread
constexpr int64_t kSmallSort = (int64_t)kListThreads * kSmallSortItems;
constexpr int64_t kSmallMax = (int64_t)kListThreads * kSmallItems;
constexpr int64_t kSmallTiles = 16384;                            // tiles whose lengths a block adds up
constexpr int64_t kSmallWork = 16 << 20;                          // Gaussians times blocks

template <int kItems>
__global__ __launch_bounds__(kListThreads) void k_small_depth_sort(const uint32_t* __restrict__ depth_key,
                                                                   const gs_splat* __restrict__ splats, int n,
                                                                   uint2* __restrict__ out)
{
    constexpr int R = kRadix, kWaves = kListThreads / kWave, kSlice = kWave * kItems;
    __shared__ uint32_t wcnt[kWaves][R];
    __shared__ uint32_t buf[kListThreads * kItems];
    __shared__ uint32_t lds16[kWaves];
    const int t = threadIdx.x, wave = t >> 6, lane = __lane_id();
    const int base = wave * kSlice + lane;
    static_assert(kListThreads * kItems <= 1 << 15, "index and rank share a register");
    uint32_t key[kItems], vr[kItems];   // vr: index | rank << 16
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int idx = base + i * kWave;
        key[i] = idx < n ? depth_key[idx] : 0u;
        vr[i] = (uint32_t)idx;
    }
#pragma unroll 1
    for (int shift = 0; shift < 32; shift += 8) {
        for (int k = t; k < kWaves * R; k += kListThreads) (&wcnt[0][0])[k] = 0;
        __syncthreads();
        // stable ranks, as in k_radix_scatter
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const bool valid = base + i * kWave < n;
            const uint32_t d = (key[i] >> shift) & (R - 1);
            const uint64_t peers = match_digit<8>(d, valid);
            const uint32_t r = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t pre = valid ? wcnt[wave][d] : 0u;
            vr[i] |= (pre + r) << 16;
            if (valid && r == 0) wcnt[wave][d] = pre + (uint32_t)__popcll(peers);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        uint32_t sum = 0, total;
        if (t < R)
            for (int w = 0; w < kWaves; ++w) sum += wcnt[w][t];
        uint32_t first = wg_excl_scan_1024(sum, lds16, &total);
        if (t < R)
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t c = wcnt[w][t];
                wcnt[w][t] = first;
                first += c;
            }
        __syncthreads();
        // the keys, then the values, through one buffer into their new places
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            if (base + i * kWave < n) {
                vr[i] += wcnt[wave][(key[i] >> shift) & (R - 1)] << 16;
                buf[vr[i] >> 16] = key[i];
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            if (base + i * kWave < n) key[i] = buf[base + i * kWave];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            if (base + i * kWave < n) buf[vr[i] >> 16] = vr[i] & 0xFFFFu;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            if (base + i * kWave < n) vr[i] = buf[base + i * kWave];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int pos = base + i * kWave;
        if (pos < n) {
            const uint2 r = splat_rect(splats, vr[i]);
            out[pos] = make_uint2(vr[i], key[i] != 0xFFFFFFFFu ? pack_rect32(r) : kEmptyRect32);
        }
    }
}

// One workgroup per block: the lengths of its 16 tile lists. Lengths need no
// order, so nothing is compacted: each wave adds up ballots of its Gaussians'
// masks in scalar registers (15 us for 20,001 Gaussians in 130 blocks, 22 with the lists
// compacted first as below; 2.9 and 4.5 for 1,024 in one).
__global__ __launch_bounds__(kListThreads) void k_small_counts(const uint2* __restrict__ order, int n, int blocks_x,
                                                               int tiles_x, int tiles_y,
                                                               uint32_t* __restrict__ tile_len)
{
    constexpr int kWaves = kListThreads / kWave, kTiles = kBlockDim * kBlockDim;
    static_assert(kWaves == kTiles && kTiles <= kWave, "a wave per tile");
    __shared__ uint32_t counts[kWaves][kTiles];
    const int t = threadIdx.x, wave = t >> 6, lane = __lane_id();
    const int bx = (int)blockIdx.x % blocks_x, by = (int)blockIdx.x / blocks_x;
    uint32_t c[kTiles] = {};
    for (int i0 = wave * kWave; i0 < n; i0 += 4 * kListThreads) {
        uint2 r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kListThreads + lane;
            r[u] = i < n ? unpack_rect32(order[i].y) : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t m = tile_mask(r[u], bx, by);
            if (__ballot(m != 0) == 0) continue;
#pragma unroll
            for (int k = 0; k < kTiles; ++k) c[k] += (uint32_t)__popcll(__ballot((m >> k) & 1u));
        }
    }
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < kTiles; ++k) mine = lane == k ? c[k] : mine;
    if (lane < kTiles) counts[wave][lane] = mine;
    __syncthreads();
    const int tx = kBlockDim * bx + (t & 3), ty = kBlockDim * by + (t >> 2);
    if (t >= kTiles || tx >= tiles_x || ty >= tiles_y) return;
    uint32_t len = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) len += counts[w][t];
    tile_len[ty * tiles_x + tx] = len;
}

// One workgroup per block, one wave per tile of it. The Gaussians that meet the
// block are compacted, in depth order, into LDS (index and mask of the block's
// tiles; indices are below kSmallMax, so both share a word); each wave then
// writes those of its tile at the sum of the lengths of the tiles before, which
// every workgroup adds up for its own four rows of tiles. Pairs over the capacity (the preprocess's count, or the
// lengths' sum) leave every range empty.
template <int kItems>
__global__ __launch_bounds__(kListThreads) void k_small_lists(const uint2* __restrict__ order, int n,
                                                              int blocks_x,
                                                              int tiles_x, int tiles_y,
                                                              const uint32_t* __restrict__ tile_len,
                                                              PairCount pairs, uint64_t capacity,
                                                              uint32_t* __restrict__ values,
                                                              uint32_t* __restrict__ tile_ids,
                                                              uint32_t* __restrict__ tile_ranges)
{
    constexpr int kWaves = kListThreads / kWave, kSlice = kWave * kItems;
    constexpr int kFly = 4;   // rounds whose loads are in flight together
    static_assert(kWaves == kBlockDim * kBlockDim, "a wave per tile");
    static_assert(kSmallMax <= 1 << 16, "index and mask share a word");
    __shared__ uint16_t smask[kListThreads * kItems];
    __shared__ uint32_t list[kListThreads * kItems];
    __shared__ uint32_t wcount[kWaves];
    __shared__ uint64_t sums[kWaves][kBlockDim + 1];
    const int t = threadIdx.x, wave = t >> 6, lane = __lane_id();
    const int bx = (int)blockIdx.x % blocks_x, by = (int)blockIdx.x / blocks_x;
    // masks of this wave's slice of the Gaussians
    uint32_t found = 0;
    const int w0 = wave * kSlice, w1 = min(w0 + kSlice, n);
    for (int i0 = w0; i0 < w1; i0 += 4 * kWave) {
        uint2 r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kWave + lane;
            r[u] = i < w1 ? unpack_rect32(order[i].y) : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kWave + lane;
            const uint32_t m = tile_mask(r[u], bx, by);
            if (i < w1) smask[i] = (uint16_t)m;
            found += (uint32_t)__popcll(__ballot(m != 0));
        }
    }
    if (lane == 0) wcount[wave] = found;
    // lengths of the tiles before each row of this block's, and of all tiles
    uint64_t s[kBlockDim + 1] = {};
    const int n_tiles = tiles_x * tiles_y;
    for (int k = t; k < n_tiles; k += kListThreads) {
        const uint32_t len = tile_len[k];
#pragma unroll
        for (int r = 0; r < kBlockDim; ++r)
            s[r] += k < (kBlockDim * by + r) * tiles_x + kBlockDim * bx ? len : 0u;
        s[kBlockDim] += len;
    }
#pragma unroll
    for (int r = 0; r <= kBlockDim; ++r) {
        for (int o = 32; o > 0; o >>= 1) s[r] += __shfl_xor(s[r], o);
        if (lane == 0) sums[wave][r] = s[r];
    }
    __syncthreads();
    uint32_t at = 0, m_all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        at += w < wave ? wcount[w] : 0u;
        m_all += wcount[w];
    }
    for (int i0 = w0; i0 < w1; i0 += kFly * kWave) {
        uint32_t gid[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const int i = i0 + u * kWave + lane;
            gid[u] = i < w1 ? order[i].x : 0u;
        }
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const int i = i0 + u * kWave + lane;
            const uint32_t m = i < w1 ? smask[i] : 0u;
            const uint64_t b = __ballot(m != 0);
            if (m != 0) list[at + (uint32_t)__popcll(b & lanemask_lt())] = gid[u] | (m << 16);
            at += (uint32_t)__popcll(b);
        }
    }
    __syncthreads();
    const int tx = kBlockDim * bx + (wave & 3), ty = kBlockDim * by + (wave >> 2);
    if (tx >= tiles_x || ty >= tiles_y) return;
    const int tile = ty * tiles_x + tx;
    uint64_t start = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        start += sums[w][wave >> 2];
        total += sums[w][kBlockDim];
    }
    for (int k = 0; k < (wave & 3); ++k) start += tile_len[tile - (wave & 3) + k];
    const bool over = pairs.overflow() || total > capacity;
    uint32_t pos = (uint32_t)start;
    for (uint32_t e0 = 0; e0 < m_all && !over; e0 += kFly * kWave) {
        uint32_t v[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const uint32_t e = e0 + u * kWave + lane;
            v[u] = e < m_all ? list[e] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const bool on = (v[u] >> (16 + wave)) & 1u;
            const uint64_t b = __ballot(on);
            if (on) {
                const uint32_t q = pos + (uint32_t)__popcll(b & lanemask_lt());
                values[q] = v[u] & 0xFFFFu;
                if (tile_ids) tile_ids[q] = (uint32_t)tile;
            }
            pos += (uint32_t)__popcll(b);
        }
    }
    if (lane == 0) {
        tile_ranges[2 * tile] = over ? 0u : (uint32_t)start;
        tile_ranges[2 * tile + 1] = over ? 0u : pos;
    }
}

}  // namespace

// Workgroups per group sum of a radix pass: the rows a workgroup adds up, group
// sums and then counts, are fewest near the square root.
int radix_group(int nblocks)
{
    int g = 1;
    while ((int64_t)g * g < nblocks) ++g;
    return g;
}

int radix_groups(int64_t keys, int tile)
{
    const int nblocks = (int)std::max<int64_t>(div_up(keys, tile), 1);
    return (int)div_up(nblocks, radix_group(nblocks));
}

// Keys per thread of the depth sort's passes (1,024 threads), of 4, 8 and 12: the
// fewest that make at most one workgroup per compute unit (256), so that no unit
// has a second one to itself; 12 for more keys than that, whose runs per digit are
// the longest. The whole binning with 4 / 8 / 12, us, at 1600x1064: 1.00M Gaussians
// 136 / 156 / 176, 1.06M 162 / 158 / 178, 2.10M (2^21) 222 / 208 / 222, 2.11M
// 248 / 253 / 226, 3M 309 / 307 / 282, 6M 559 / 513 / 495. Scatters at 6M: 290 with
// 8, 273 with 12, 319 with 16, which spill. (Rectangles gathered, on grids beyond
// 256 tiles a side: the same lines; 12 with 8M and more is 3% behind workgroups of
// 4,096 keys, 588 against 568.)
int depth_items(int64_t n) { return n <= (1 << 20) ? 4 : n <= (1 << 21) ? 8 : 12; }

// Depth sort of the n Gaussians and their tile rectangles. On grids of at most
// 256 x 256 tiles the rectangles travel with the sort in 32 bits, read from the
// records in index order by the first pass: 4 bytes more per Gaussian and pass,
// where the last pass would otherwise gather one 128-byte line per Gaussian
// (60 us of that pass's 78 at 3M Gaussians, 155 at 6M).
bool packed_rects(const Cam& cam) { return cam.tiles_x <= 256 && cam.tiles_y <= 256; }

template <int kItems>
static void depth_passes(const Cam& cam, int64_t n, const uint32_t* depth_key, const gs_splat* splats,
                         const Workspace& ws, DepthOrder* out, hipStream_t s)
{
    uint32_t* kbuf[2] = {ws.keys_a, ws.keys_b};
    const PairCount keys_n{nullptr, (uint64_t)n, (uint64_t)n};
    const int groups = radix_groups(n, kListThreads * kItems);
    auto sup = [&](int p) { return ws.depth_sup + (size_t)p * groups * kRadix; };
    *out = DepthOrder{nullptr, nullptr, nullptr};
    if (packed_rects(cam)) {
        uint2* vbuf[2] = {ws.vals_a, ws.vals_b};
        radix_pass<8, kItems, uint2, kFirst>(depth_key, nullptr, keys_n, 0, kbuf[0], vbuf[0], ws.hist, sup(0), s,
                                             splats);
        for (int p = 1; p < 4; ++p)
            radix_pass<8, kItems, uint2, kPlain>(kbuf[(p & 1) ^ 1], vbuf[(p & 1) ^ 1], keys_n, 8 * p,
                                                 p == 3 ? nullptr : kbuf[p & 1], vbuf[p & 1], ws.hist, sup(p), s);
        out->packed = vbuf[1];
    } else {
        // indices alone: both buffers in one of the pair buffers, the rectangles in the other
        uint32_t* vbuf[2] = {reinterpret_cast<uint32_t*>(ws.vals_a), reinterpret_cast<uint32_t*>(ws.vals_a) + n};
        for (int p = 0; p < 3; ++p)
            radix_pass<8, kItems, uint32_t, kPlain>(p == 0 ? depth_key : kbuf[(p & 1) ^ 1],
                                                    p == 0 ? nullptr : vbuf[(p & 1) ^ 1], keys_n, 8 * p, kbuf[p & 1],
                                                    vbuf[p & 1], ws.hist, sup(p), s);
        radix_pass<8, kItems, uint32_t, kGather>(kbuf[0], vbuf[0], keys_n, 24, nullptr, vbuf[1], ws.hist, sup(3), s,
                                                 splats, ws.vals_b);
        out->gid = vbuf[1];
        out->rect = ws.vals_b;
    }
}

int blocks_x_of(const Cam& cam) { return (cam.tiles_x + kBlockDim - 1) / kBlockDim; }
int blocks_y_of(const Cam& cam) { return (cam.tiles_y + kBlockDim - 1) / kBlockDim; }
int64_t segment_bound(const Cam& cam, uint64_t capacity)
{
    return div_up((int64_t)capacity, kSegEntries) + (int64_t)blocks_x_of(cam) * blocks_y_of(cam);
}

hipError_t launch_entry_offsets(int64_t n, PairCount pairs, const DepthOrder& order, const Workspace& ws,
                                hipStream_t s)
{
    const int nb = (int)div_up(n, kDupChunk);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(kBlock), 0, s, order, n, ws.scan_part);
    };
    if (order.packed) launch(k_entry_partial<true>);
    else launch(k_entry_partial<false>);
    if (nb > kSumChunks)
        hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kBlock), 0, s, ws.scan_part, nb, pairs, ws.entry_count);
    return hipGetLastError();
}

// Bits of the block id.
static int block_bits(const Cam& cam)
{
    const uint32_t nb = (uint32_t)blocks_x_of(cam) * (uint32_t)blocks_y_of(cam);
    int bits = 0;
    while (bits < 32 && ((nb - 1) >> bits) != 0) ++bits;
    return bits;
}

bool blocks_supported(const Cam& cam) { return block_bits(cam) <= 32 - kMaskBits; }

hipError_t launch_block_entries(const Cam& cam, int64_t n, const DepthOrder& order, PairCount pairs,
                                uint64_t capacity, const Workspace& ws, hipStream_t s)
{
    const int nb = (int)div_up(n, kDupChunk);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(kBlock), 0, s, order, n, ws.scan_part, blocks_x_of(cam),
                           pairs, capacity, ws.entry_count, ws.entry_keys_a, ws.entry_vals_a);
    };
    const bool sum = nb <= kSumChunks;
    if (order.packed) sum ? launch(k_block_entries<true, true>) : launch(k_block_entries<true, false>);
    else sum ? launch(k_block_entries<false, true>) : launch(k_block_entries<false, false>);
    return hipGetLastError();
}

// Stable LSD sort of the entries by block id, the key bits above the tile
// mask (passes of <= 9 bits; none with a single block), then each block's
// entry range (the digit totals of a single pass, else a search of the sorted
// keys) and the segment table.
hipError_t launch_block_sort(const Cam& cam, PairCount entries, const Workspace& ws, BlockEntries* out, hipStream_t s)
{
    const int n_blocks = blocks_x_of(cam) * blocks_y_of(cam);
    const int bits = block_bits(cam);
    const int passes = (bits + kBlockSortBits - 1) / kBlockSortBits;
    const int items = block_items(entries.host);
    uint32_t* kbuf[2] = {ws.entry_keys_a, ws.entry_keys_b};
    uint32_t* vbuf[2] = {ws.entry_vals_a, ws.entry_vals_b};
    int src = 0, shift = kMaskBits;
    // a single pass's digit totals are the blocks' entry counts: its scatter's
    // extra workgroup writes the segment table
    const SegTable seg_one{ws.block_ranges, ws.seg_base, ws.seg_block, ws.list_counters, n_blocks};
    const SegTable seg_none{nullptr, nullptr, nullptr, nullptr, 0};
    for (int p = 0; p < passes; ++p) {
        const int pb = (kMaskBits + bits - shift + (passes - p) - 1) / (passes - p);   // remaining bits spread evenly
        uint32_t* sup = ws.block_sup + (size_t)p * radix_groups((int64_t)entries.host, kListThreads * items) * 2 * kRadix;
        auto pass = items == kBlockSortItems ? block_radix_pass<kBlockSortItems> : block_radix_pass<2 * kBlockSortItems>;
        const hipError_t e = pass(kbuf[src], vbuf[src], entries, shift, pb, kbuf[src ^ 1], vbuf[src ^ 1], ws.hist, sup,
                                  s, passes == 1 ? seg_one : seg_none);
        if (e != hipSuccess) return e;
        shift += pb;
        src ^= 1;
    }
    if (passes != 1) {   // none (a single block) or several: ranges by search, then the table
        const dim3 grid((unsigned)div_up(n_blocks + 1, kBlock / kWave));
        hipLaunchKernelGGL(k_ranges, grid, dim3(kBlock), 0, s, kbuf[src], kMaskBits, entries, n_blocks,
                           ws.block_ranges);
        hipLaunchKernelGGL(k_segments, dim3(1), dim3(kListThreads), 0, s, seg_one);
    }
    out->key = kbuf[src];
    out->gid = vbuf[src];
    return hipGetLastError();
}

hipError_t launch_tile_lists(const Cam& cam, PairCount pairs, uint64_t capacity, const Workspace& ws,
                             const BlockEntries& ent, uint32_t* values, uint32_t* tile_ids, uint32_t* tile_ranges,
                             hipStream_t s)
{
    const int bx = blocks_x_of(cam), n_blocks = bx * blocks_y_of(cam);
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    const dim3 segs((unsigned)segment_bound(cam, capacity));
    hipLaunchKernelGGL(k_tile_count, segs, dim3(kBlock), 0, s, ent.key, ws.block_ranges, ws.seg_base, ws.seg_block,
                       ws.list_counters, ws.seg_cnt);
    hipLaunchKernelGGL(k_tile_scan, dim3(n_blocks), dim3(kWave), 0, s, ws.seg_base, n_blocks, bx, cam.tiles_x,
                       cam.tiles_y, ws.seg_cnt, tile_ranges);
    hipLaunchKernelGGL(k_tile_starts, dim3(1), dim3(kListThreads), 0, s, n_tiles, pairs, capacity, tile_ranges,
                       ws.list_counters);
    if (tile_ids)
        hipLaunchKernelGGL(k_tile_emit<true>, segs, dim3(kBlock), 0, s, ent.key, ent.gid, ws.block_ranges,
                           ws.seg_base, ws.seg_block, ws.list_counters, bx, cam.tiles_x, ws.seg_cnt, tile_ranges,
                           values, tile_ids);
    else
        hipLaunchKernelGGL(k_tile_emit<false>, segs, dim3(kBlock), 0, s, ent.key, ent.gid, ws.block_ranges,
                           ws.seg_base, ws.seg_block, ws.list_counters, bx, cam.tiles_x, ws.seg_cnt, tile_ranges,
                           values, tile_ids);
    return hipGetLastError();
}

// Whether the tile lists come from small_lists: within its LDS, and where the
// blocks' search of all Gaussians costs less than the launches it saves (up to
// kSmallWork tests). Each workgroup compacts every Gaussian that it finds, so with
// more than kSmallSort of them there has to be work for many: a block for every
// kListThreads Gaussians (the whole binning this way / with block entries, us, lists
// of a few and of all Gaussians: 16,384 in 1 block 97 to 99 / 79 to 81, in 12
// 81 and 99 / 87 and 101, in 35 79 and 101 / 92 and 132; 24,576 in 1 block 118 to 121 / 80 to 82,
// in 12 94 and 121 / 90 and 105, in 35 88 and 122 / 93 and 136).
bool small_lists(const Cam& cam, int64_t n)
{
    const int64_t blocks = (int64_t)blocks_x_of(cam) * blocks_y_of(cam);
    return n <= kSmallMax && packed_rects(cam) && (int64_t)cam.tiles_x * cam.tiles_y <= kSmallTiles &&
           n * blocks <= kSmallWork && (n <= kSmallSort || n <= blocks * kListThreads);
}

template <int kItems>
static void small_depth(int n, const uint32_t* depth_key, const gs_splat* splats, uint2* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_small_depth_sort<kItems>, dim3(1), dim3(kListThreads), 0, s, depth_key, splats, n, out);
}

template <int kItems>
static void small_tiles(const Cam& cam, int n, const uint2* order, PairCount pairs, uint64_t capacity,
                        uint32_t* tile_len, uint32_t* values, uint32_t* tile_ids, uint32_t* tile_ranges, hipStream_t s)
{
    const int bx = blocks_x_of(cam);
    const dim3 blocks((unsigned)(bx * blocks_y_of(cam)));
    hipLaunchKernelGGL(k_small_counts, blocks, dim3(kListThreads), 0, s, order, n, bx, cam.tiles_x, cam.tiles_y,
                       tile_len);
    hipLaunchKernelGGL(k_small_lists<kItems>, blocks, dim3(kListThreads), 0, s, order, n, bx, cam.tiles_x,
                       cam.tiles_y, tile_len, pairs, capacity, values, tile_ids, tile_ranges);
}

hipError_t launch_small_lists(const Cam& cam, int64_t n, const DepthOrder& order, PairCount pairs, uint64_t capacity,
                              const Workspace& ws, uint32_t* values, uint32_t* tile_ids, uint32_t* tile_ranges,
                              hipStream_t s)
{
    auto f = n <= kListThreads ? small_tiles<1> : n <= 4 * kListThreads ? small_tiles<4>
             : n <= 12 * kListThreads ? small_tiles<12> : small_tiles<kSmallItems>;
    f(cam, (int)n, order.packed, pairs, capacity, ws.walk_cls, values, tile_ids, tile_ranges, s);
    return hipGetLastError();
}

bool small_depth_sort(const Cam& cam, int64_t n) { return n <= kSmallSort && packed_rects(cam); }

hipError_t launch_clear_sums(const Workspace& ws, hipStream_t s)
{
    return launch_fill_u32(ws.depth_sup, ws.sup_count, 0u, s);   // the block sort's lie behind the depth sort's
}

hipError_t launch_depth_sort(const Cam& cam, int64_t n, const uint32_t* depth_key, const gs_splat* splats,
                             const Workspace& ws, DepthOrder* out, hipStream_t s)
{
    if (small_depth_sort(cam, n)) {
        auto f = n <= kListThreads ? small_depth<1> : n <= 2 * kListThreads ? small_depth<2>
                 : n <= 4 * kListThreads ? small_depth<4> : n <= 8 * kListThreads ? small_depth<8>
                 : small_depth<kSmallSortItems>;
        f((int)n, depth_key, splats, ws.vals_b, s);
        *out = DepthOrder{ws.vals_b, nullptr, nullptr};
        return hipGetLastError();
    }
    switch (depth_items(n)) {
    case 4: depth_passes<4>(cam, n, depth_key, splats, ws, out, s); break;
    case 8: depth_passes<8>(cam, n, depth_key, splats, ws, out, s); break;
    default: depth_passes<12>(cam, n, depth_key, splats, ws, out, s); break;
    }
    return hipGetLastError();
}

}  // namespace gsr
