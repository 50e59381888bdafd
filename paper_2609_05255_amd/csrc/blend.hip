// Tile blend (Sec. 3.1) and its reverse. A 16x16 tile is covered by 4/PIX
// independent wave64s (PIX = 2 in the forward, 4 in the backward, fewer where an
// image has few tiles); wave w owns
// the 4 PIX contiguous rows from 4 PIX w, and every lane PIX pixels of one
// column (rows 4k apart), so a lane's pixels share dx and the quadratic form
// costs two fused multiply-adds per pixel. Each wave walks the tile's
// depth-sorted list in batches of 64 splats: every lane gathers one record
// (the next batch is fetched while the current one is blended) and tests it
// against the wave's pixels, the batch is staged in the wave's own LDS slot,
// and each splat that passes is then read back by the whole wave from one
// address (a broadcast read). No workgroup barriers; a wave stops when its own
// pixels are done. The forward takes 0.155 ms on the 3M-Gaussian 1600x1064 scene
// (0.182 ms before the alpha test moved to logarithms, the constants to the
// staging lane and the end-of-walk test to scalar lane masks).
//
// Workgroup ids are mapped to tiles so that each XCD (workgroups are dealt
// round-robin over the 8 XCDs) renders a contiguous band of tiles, whose lists
// share most splats in that XCD's L2; the backward of images up to 32768 tiles
// takes them longest walk first instead (the tile order below).
#include "gs_internal.h"

namespace gsr {

namespace {

constexpr int kXcds = 8;

// Pixels per lane (1, 2 or 4: four, two or one wave per tile), by the number of
// tiles. Few tiles leave the SIMDs (1,024) short of waves, and the kernel lasts
// as long as its longest walk: more waves per tile shorten each, at the price of
// each splat's set-up and reduction once per wave. The lines lie where both
// sides measure equal over lists of small and of large splats (the whole backward,
// us, 1 / 2 / 4 pixels per lane, 20,000 Gaussians of 2 to 18 tiles each and 8,192 of
// 8 to 240):
//   64 tiles   270 / 408 / 772 and 95 / 120 / 184,
//   475 tiles   95 / 138 / 220 and 56 / 71 / 101,
//   1200 tiles  80 / 106 / 166 and 75 / 68 / 90,
//   1536 tiles  78 / 99 / 151 and 83 / 80 / 88,
//   1900 tiles  78 / 99 / 149 and 93 / 82 / 88,
//   3072 tiles  92 / 93 / 134 and 128 / 106 / 96
// and the forward kernel: 64 tiles 43 / 75, 600 tiles 62 / 89, 1200 tiles 62 / 76,
//   1900 tiles 87 / 90, 2560 tiles 91 / 92, 3200 tiles 121 / 115
inline int fwd_pix(int n_tiles) { return n_tiles <= 2048 ? 1 : 2; }
inline int bwd_pix(int n_tiles) { return n_tiles <= 1536 ? 1 : n_tiles <= 3072 ? 2 : 4; }

// Splats per step of the walks with one pixel per lane: a wave nearly alone on
// its SIMD waits for each splat's LDS reads and exponential, which a step's
// splats share (64 tiles: forward 56 us with one, 52 with two, 43 with four,
// backward 77, 75 and 76).
constexpr int kFwdGroup = 4, kBwdGroup = 2;

__device__ __forceinline__ int tile_of_block(int block, int n_tiles)
{
    const int per = (n_tiles + kXcds - 1) / kXcds;
    return (block % kXcds) * per + block / kXcds;
}

inline int blend_grid(int n_tiles) { return (int)div_up(n_tiles, kXcds) * kXcds; }

constexpr float kAlphaMax = 0.99f;
constexpr float kTMin = 0.0001f;
constexpr float kLog2e = 1.4426950408889634f;


// A splat as the walks read it from LDS: the record with the constants of the
// quadratic form taken once by the lane that stages it. In base-2 units (times
// log2 e), so that exp(power) is one hardware exp2: with k = log2(e) / 2,
// -power log2 e = k (ca dx^2 + cb2 dx dy) + kc dy^2 with cb2 = 2 b and kc = k c.
// k goes with dx (column_quad), where its rounding differs from column to column.
// Staged with the conic (k a, 2 k b) it is the same at every pixel of a splat and
// adds up: for splats of sigma 60 x 0.5 pixels under a smooth upstream gradient the
// error of the opacity's gradient was 2.5 times as large (1.1e-5 to 2.8e-5 of it, now
// 0.5e-5 to 1.1e-5), for one vector instruction less per visit of the forward (no
// time measured: a paper-scale render 663 us either way). e_max is the bound of
// -power log2 e where alpha reaches 1/255, log2(255 opacity).
struct Staged {
    float mx, my, ca, cb2, kc, op, r, g, b, e_max;
};

__device__ __forceinline__ void stage_words(const float4& c0, const float4& c1, const float4& c2, float4& w0,
                                            float4& w1, float2& w2)
{
    w0 = make_float4(c0.x, c0.y, c0.z, 2.f * c0.w);
    w1 = make_float4((0.5f * kLog2e) * c1.x, c1.y, c1.z, c1.w);
    // the hardware logarithm corrected by the residual of its exponential. Over all
    // opacities above 1/255 it is within 3.9e-7 of log2(255 o), and within 1.9e-7
    // below 2/255 (measured): 2.7e-7 and 1.3e-7 of alpha. The hardware exponential
    // and the product of o e^power >= 1/255 are within 1.8e-7, so the test decides
    // about as closely on the logarithms.
    const float r255 = 255.f * c1.y;
    const float l = __builtin_amdgcn_logf(r255);
    const float reach = __fmaf_rn(__fmaf_rn(r255, __builtin_amdgcn_exp2f(-l), -1.f), kLog2e, l);
    w2 = make_float2(c2.x, reach > 0.f ? reach : 0.f);
}

__device__ __forceinline__ Staged staged(const float4& w0, const float4& w1, const float2& w2)
{
    return Staged{w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w, w2.x, w2.y};
}

// The backward needs the record's b and c as well, for the gradient of the mean:
// in the third plane's spare words.
struct StagedBwd : Staged {
    float cb, cc;
};

__device__ __forceinline__ void stage_words_bwd(const float4& c0, const float4& c1, const float4& c2, float4& w0,
                                                float4& w1, float4& w2)
{
    float2 tail;
    stage_words(c0, c1, c2, w0, w1, tail);
    w2 = make_float4(tail.x, tail.y, c0.w, c1.x);
}

__device__ __forceinline__ StagedBwd staged_bwd(const float4& w0, const float4& w1, const float4& w2)
{
    return StagedBwd{staged(w0, w1, make_float2(w2.x, w2.y)), w2.z, w2.w};
}

// A wave's staged batch: three planes at one 16-byte stride, so that a splat's
// reads share one address register.
struct StageSlot {
    float4 w[3][kWave];
    __device__ __forceinline__ float2& tail(int j) { return reinterpret_cast<float2&>(w[2][j]); }
};

// -power log2 e of one column as a polynomial in dy: q0 + dy (q1 + dy kc).
struct Quad {
    float q0, q1;
};

__device__ __forceinline__ Quad column_quad(const Staged& s, float dx)
{
    const float kdx = (0.5f * kLog2e) * dx;
    return Quad{s.ca * dx * kdx, s.cb2 * kdx};
}

__device__ __forceinline__ float quad_neg_power(const Staged& s, const Quad& q, float dy)
{
    return __fmaf_rn(__fmaf_rn(s.kc, dy, q.q1), dy, q.q0);
}

// power <= 0 and alpha >= 1/255 (o e^power >= 1/255, on the logarithms) as one
// unsigned comparison of bit patterns: e = -power log2 e and its bound are
// non-negative where the test passes, so their bits order as their values; a
// negative e (power > 0) or a NaN has larger bits than any bound. e is never
// -0 (a > 0, so q0 is +0 or more, and sums that cancel round to +0), nor is the
// bound. Taken on the logarithm the alpha test needs no exponential, and the
// pixels that pass need no second test: 2 vector instructions fewer per pixel.
__device__ __forceinline__ bool in_reach(float e, float e_max)
{
    return __float_as_uint(e) <= __float_as_uint(e_max);
}

template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xF, 0xF, true));
}

// a's sum over the lane halves in lanes 0..31, b's in lanes 32..63 (each lane
// with its partner 32 lanes away), and the same for odd and even rows of 16.
__device__ __forceinline__ float merge32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float merge16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// dL/dmean of one splat over a lane's pixels, from their sums p0 and p1 of
// dL/dpower times 1 and dy (they share dx): (a dx p0 + b p1, c p1 + b dx p0).
// For long thin splats the two terms cancel by up to the conic's condition
// number, so they are combined here, where they are small: from the finished
// sums over all pixels (kept raw and combined once per Gaussian) the gradient's
// error was 3 to 10 times larger (5e-6 to 9e-6 of it against 0.8e-6 to 2e-6 for
// splats of sigma 40 x 4 pixels under a smooth upstream gradient, 4e-3 to 7e-3
// against 1e-3 to 2e-3 at 300 x 0.1), and it took a conic other than the blended
// record's. 5 vector instructions per visit; with column_quad's fourth product
// they are 4% of the backward's time at 3M Gaussians.
__device__ __forceinline__ void mean_terms(const StagedBwd& s, float dx, float p0, float p1, float& gx, float& gy)
{
    const float m_x = dx * p0;
    gx = __fmaf_rn(s.ca, m_x, s.cb * p1);
    gy = __fmaf_rn(s.cc, p1, s.cb * m_x);
}

// Wave sums of one splat's nine accumulator entries (kAccStride) from its eight
// per-lane sums over the lane's pixels: p0, p1, p2 (dL/dpower times 1, dy, dy^2),
// the mean's gradient (gx, gy) and the colour's c. dx is the same in the four
// lanes of a column, so the four rows of 16 lanes are added first, two values
// merged per lane swap, and the other moments in dx are products of the column
// sums. Within the rows, DPP sums take two registers (8 lanes each) and a third
// (every other quad) at once. The sum of entry e ends in lane
// reduce_src_lane(e). About 25 vector instructions, where a butterfly of selects
// and permutes over nine values took 46. Every lane of the wave must call it (a
// disabled DPP source lane reads 0).
__device__ __forceinline__ float wave_reduce9(float p0, float p1, float p2, float gx, float gy, float c0, float c1,
                                              float c2, float dx, bool upper, bool hi8, bool odd4)
{
    const float s1 = merge16(merge32(p0, p1), merge32(c0, c1));   // rows: p0, c0, p1, c1
    const float s2 = merge16(merge32(gx, gy), merge32(p2, c2));   // rows: gx, p2, gy, c2
    const float dx1 = dx * s1;
    const float dx2 = dx * dx1;
    const float s3 = upper ? dx1 : dx2;                           // row 0: p0 dx^2, row 2: p1 dx
    const float h1 = s1 + dpp_f32<0x128>(s1), h2 = s2 + dpp_f32<0x128>(s2), h3 = s3 + dpp_f32<0x128>(s3);   // row_ror:8
    const float h = hi8 ? h2 : h1;
    // both sums before the select: a select over the sums' own code would become
    // a branch that disables half of the source lanes
    const float m = h + dpp_f32<0x141>(h), m3 = h3 + dpp_f32<0x141>(h3);      // row_half_mirror
    const float q = odd4 ? m3 : m;
    const float t = q + dpp_f32<0xB1>(q);                                     // quad_perm, lane ^ 1
    return t + dpp_f32<0x4E>(t);                                              // lane ^ 2
}

// row[lane] += v with a wave-uniform row: its address is kept in scalar
// registers (folded into the lane's, it is a 64-bit vector multiply-add).
__device__ __forceinline__ void add_scalar_row(float* row, int lane, float v)
{
    uint64_t base = reinterpret_cast<uint64_t>(row);
    asm("" : "+s"(base));
    auto* p = reinterpret_cast<__attribute__((address_space(1))) float*>(base);
    __hip_atomic_fetch_add(p + lane, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kReduceLane[kAccStride] = {0, 8, 40, 4, 36, 24, 16, 48, 56};

// The lane whose sum is entry e: M0, mean x, mean y, Mxx, Mxy, Myy, c0, c1, c2.
__device__ __forceinline__ int reduce_src_lane(int e)
{
    int r = 0;
#pragma unroll
    for (int k = 0; k < kAccStride; ++k) r = e == k ? kReduceLane[k] : r;
    return r;
}

// The entry whose sum is in this lane, or -1.
__device__ __forceinline__ int reduce_entry(int lane)
{
    int r = -1;
#pragma unroll
    for (int k = 0; k < kAccStride; ++k) r = lane == kReduceLane[k] ? k : r;
    return r;
}

// Whether the splat's alpha >= 1/255 region (power >= power_min, i.e. the
// conic's quadratic form q(u, v) = a u^2 + 2 b u v + c v^2 at most
// r2 = -2 power_min) meets the box [x_lo, x_hi] x [y_lo, y_hi] of the wave's
// pixel centres. The least q over the box is 0 when the mean lies inside it,
// else it is on an edge, where q is a parabola in the free coordinate: its
// vertex, clamped to the edge. The margin, 1e-3 plus 1e-5 of the largest sum
// of the three terms' magnitudes over the box, is far above the rounding of
// this evaluation and of the per-pixel power (a few ulp of that sum), so a
// splat found apart from the box reaches power_min at none of its pixels.
__device__ __forceinline__ bool ellipse_meets_box(float mx, float my, float a, float b, float c, float pmin,
                                                  float x_lo, float x_hi, float y_lo, float y_hi)
{
    const float r2 = -2.f * pmin;
    const float u0 = x_lo - mx, u1 = x_hi - mx, v0 = y_lo - my, v1 = y_hi - my;
    const float ia = __builtin_amdgcn_rcpf(a), ic = __builtin_amdgcn_rcpf(c);
    auto q = [&](float u, float v) { return a * u * u + 2.f * b * u * v + c * v * v; };
    auto on_u = [&](float u) { return q(u, fminf(fmaxf(-b * u * ic, v0), v1)); };   // edge of fixed u
    auto on_v = [&](float v) { return q(fminf(fmaxf(-b * v * ia, u0), u1), v); };   // edge of fixed v
    const bool inside = u0 <= 0.f && u1 >= 0.f && v0 <= 0.f && v1 >= 0.f;
    const float qmin = inside ? 0.f : fminf(fminf(on_u(u0), on_u(u1)), fminf(on_v(v0), on_v(v1)));
    const float um = fmaxf(fabsf(u0), fabsf(u1)), vm = fmaxf(fabsf(v0), fabsf(v1));
    const float terms = a * um * um + c * vm * vm + 2.f * fabsf(b) * um * vm;
    return qmin <= r2 + (1e-3f + 1e-5f * terms);
}

}  // namespace

template <int kPix>
__global__ __launch_bounds__(kTile * kTile / kPix) void k_blend_fwd(Cam cam, const gs_splat* __restrict__ splats,
                                                                    const uint32_t* __restrict__ values,
                                                                    const uint32_t* __restrict__ ranges,
                                                                    float* __restrict__ image,
                                                                    float* __restrict__ final_T,
                                                                    uint32_t* __restrict__ n_contrib)
{
    constexpr int kRowStep = 4;   // pixel k of a lane lies 4k rows below its first
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    const int tile = tile_of_block(blockIdx.x, n_tiles);
    if (tile >= n_tiles) return;
    const int lane = __lane_id();
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    // wave w covers the 4 kPix contiguous rows starting at 4 kPix w
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x = tx * kTile + (lane & 15);
    const int y0 = ty * kTile + 4 * kPix * wave + (lane >> 4);
    const float px = (float)x + 0.5f;
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
    // box of this wave's pixel centres: 16 columns, 4 kPix rows
    const float box_cx = (float)(tx * kTile) + 8.f, box_hx = 7.5f;
    const float box_lo = (float)(ty * kTile + 4 * kPix * wave) + 0.5f;
    const float box_hi = box_lo + (float)(4 * kPix - 1);
    const float box_cy = 0.5f * (box_lo + box_hi), box_hy = 0.5f * (box_hi - box_lo);

    // T > 0 while the pixel still blends; the stop rule (and a pixel outside
    // the image) makes it negative, |T| keeping the final transmittance
    float T[kPix], C0[kPix], C1[kPix], C2[kPix], py[kPix];
    uint32_t last[kPix];
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        C0[k] = C1[k] = C2[k] = 0.f;
        last[k] = 0;
        py[k] = (float)(y0 + kRowStep * k) + 0.5f;
        T[k] = (x < cam.width && (y0 + kRowStep * k) < cam.height) ? 1.f : -1.f;
    }
    uint64_t alive = 0;   // lanes with a pixel still blending
#pragma unroll
    for (int k = 0; k < kPix; ++k) alive |= __ballot(T[k] > 0.f);
    // each batch of 64 list entries is staged in LDS; the wave then reads one
    // record per step at a uniform address (a broadcast read: no vector
    // instructions, unlike a lane-by-lane readlane broadcast)
    __shared__ StageSlot stage[kTile * kTile / kPix / kWave];
    StageSlot& st = stage[wave];
    float4 c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0, c2 = c0;
    if (start + lane < end) {
        const float4* p = reinterpret_cast<const float4*>(splats + values[start + lane]);
        c0 = p[0]; c1 = p[1]; c2 = p[2];
    }
    // the list entry of the batch after the prefetched one, loaded a batch early
    uint32_t nid = start + kWave + lane < end ? values[start + kWave + lane] : 0u;
    for (uint32_t b = start; b < end && alive != 0; b += kWave) {
        stage_words(c0, c1, c2, st.w[0][lane], st.w[1][lane], st.tail(lane));
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // skip the splats that reach alpha >= 1/255 nowhere in this wave's
        // pixels: each lane tests the record it holds (before the next batch
        // replaces it; the bounding box first, then the ellipse), and the walk
        // below visits only the others, in order
        const int cnt = (int)min((uint32_t)kWave, end - b);
        const bool meets = lane < cnt && fabsf(c0.x - box_cx) <= c2.z + box_hx &&
                           fabsf(c0.y - box_cy) <= c2.w + box_hy &&
                           ellipse_meets_box(c0.x, c0.y, c0.z, c0.w, c1.x, c2.y, box_cx - box_hx, box_cx + box_hx,
                                             box_lo, box_hi);
        uint64_t todo = __ballot(meets);
        if (b + kWave + lane < end) {
            const float4* p = reinterpret_cast<const float4*>(splats + nid);
            c0 = p[0]; c1 = p[1]; c2 = p[2];
        }
        if (b + 2 * kWave + lane < end) nid = values[b + 2 * kWave + lane];
        if constexpr (kPix == 1) {
            // few tiles: a step takes kFwdGroup splats, whose reads and exponentials
            // overlap, without branches; only the transmittance goes from one to
            // the next (the same operations per pixel as below)
            while (todo != 0) {
                Staged s[kFwdGroup];
                float alpha[kFwdGroup];
                uint32_t pos[kFwdGroup];
                uint64_t in[kFwdGroup];
                int j = 0;
#pragma unroll
                for (int g = 0; g < kFwdGroup; ++g) {
                    const uint64_t some = todo != 0 ? ~0ull : 0ull;   // none left: the last one again, masked out
                    j = todo != 0 ? (int)__builtin_ctzll(todo) : j;
                    todo &= todo - 1;
                    s[g] = staged(st.w[0][j], st.w[1][j], st.tail(j));
                    pos[g] = b - start + (uint32_t)j + 1;
                    in[g] = some;
                }
#pragma unroll
                for (int g = 0; g < kFwdGroup; ++g) {
                    const float e = quad_neg_power(s[g], column_quad(s[g], px - s[g].mx), py[0] - s[g].my);
                    in[g] &= __ballot(in_reach(e, s[g].e_max));
                    alpha[g] = fminf(kAlphaMax, s[g].op * __builtin_amdgcn_exp2f(-e));
                }
#pragma unroll
                for (int g = 0; g < kFwdGroup; ++g) {
                    const bool on = __builtin_amdgcn_inverse_ballot_w64(in[g] & __ballot(T[0] > 0.f));
                    const float Tn = T[0] * (1.f - alpha[g]);
                    const bool stop = Tn < kTMin;
                    const float w = stop ? 0.f : alpha[g] * T[0];
                    C0[0] = on ? __fmaf_rn(s[g].r, w, C0[0]) : C0[0];
                    C1[0] = on ? __fmaf_rn(s[g].g, w, C1[0]) : C1[0];
                    C2[0] = on ? __fmaf_rn(s[g].b, w, C2[0]) : C2[0];
                    last[0] = on && !stop ? pos[g] : last[0];
                    T[0] = on ? (stop ? -T[0] : Tn) : T[0];
                }
                alive = __ballot(T[0] > 0.f);
                if (alive == 0) break;
            }
        } else {
            while (todo != 0) {
                const int j = (int)__builtin_ctzll(todo);
                todo &= todo - 1;
                const Staged s = staged(st.w[0][j], st.w[1][j], st.tail(j));
                const float dx = px - s.mx;
                const Quad q = column_quad(s, dx);
                alive = 0;
#pragma unroll
                for (int k = 0; k < kPix; ++k) {
                    // one branch per pixel; the stop rule is a select inside it
                    const float e = quad_neg_power(s, q, py[k] - s.my);
                    const bool on = T[k] > 0.f;
                    alive |= __ballot(on);
                    if (on & in_reach(e, s.e_max)) {
                        const float alpha = fminf(kAlphaMax, s.op * __builtin_amdgcn_exp2f(-e));
                        const float Tn = T[k] * (1.f - alpha);
                        const bool stop = Tn < kTMin;
                        const float w = stop ? 0.f : alpha * T[k];
                        C0[k] = __fmaf_rn(s.r, w, C0[k]);
                        C1[k] = __fmaf_rn(s.g, w, C1[k]);
                        C2[k] = __fmaf_rn(s.b, w, C2[k]);
                        last[k] = stop ? last[k] : b - start + (uint32_t)j + 1;
                        T[k] = stop ? -T[k] : Tn;
                    }
                }
                // no pixel was still blending before this splat (found one visit late:
                // the comparisons are those of the branches above)
                if (alive == 0) break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    const int64_t hw = (int64_t)cam.width * cam.height;
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        const int y = y0 + kRowStep * k;
        if (x >= cam.width || y >= cam.height) continue;
        const int64_t pix = (int64_t)y * cam.width + x;
        const float Tf = fabsf(T[k]);
        image[pix] = __fmaf_rn(Tf, cam.bg[0], C0[k]);
        image[hw + pix] = __fmaf_rn(Tf, cam.bg[1], C1[k]);
        image[2 * hw + pix] = __fmaf_rn(Tf, cam.bg[2], C2[k]);
        final_T[pix] = Tf;
        n_contrib[pix] = last[k];
    }
}

hipError_t launch_blend_fwd(const Cam& cam, const gs_splat* splats, const uint32_t* values,
                            const uint32_t* tile_ranges, float* image, float* final_T, uint32_t* n_contrib,
                            hipStream_t s)
{
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    auto launch = [&](auto kernel, int pix) {
        hipLaunchKernelGGL(kernel, dim3(blend_grid(n_tiles)), dim3(kTile * kTile / pix), 0, s, cam, splats, values,
                           tile_ranges, image, final_T, n_contrib);
    };
    if (fwd_pix(n_tiles) == 1) launch(k_blend_fwd<1>, 1);
    else launch(k_blend_fwd<2>, 2);
    return hipGetLastError();
}

// ---- backward -----------------------------------------------------------------
// Per pixel, back to front from its last blended splat, with T recovered as
// T_i = T_{i+1} / (1 - alpha_i) and A the composited colour behind the splat,
// projected on the upstream gradient g (A_i = A_{i+1} + alpha_i (c_i . g -
// A_{i+1}), the background at the back):  dL/dcolour_i = alpha_i T_i g,
// dL/dalpha_i = T_i (c_i . g - A_{i+1}). The alpha and skip decisions reuse the
// forward's code, so the same splats are found contributing. Each lane sums its
// pixels' terms, the wave its lanes (wave_reduce9), and a tile issues one set of
// nine float atomics per splat: its one wave by itself, several after their sums
// met in LDS.
//
// Bound by vector instruction issue: on the 3M-Gaussian 1600x1064 scene it takes
// 0.277 ms, of which its instructions alone (156M wave instructions at 4 cycles;
// the two transcendentals per pixel take 16) fill 0.25 ms or more. What shortened it
// (from 0.318 ms and 204M): second moments summed raw and their factors applied once
// per Gaussian later, no opacity sum (dL/dopacity follows from the zeroth moment),
// the recursion in A (no division beside T's), the alpha test on logarithms,
// constants taken by the staging lane, lane masks combined as scalars, scalar
// atomic addresses, and fewer instructions in the reduction.

// The sums of a tile's waves over a span of kRows list entries, one entry per
// thread of the workgroup, so that a tile issues one set of atomics per splat
// whatever its number of waves. Splats that many tiles share (a scene's first,
// large ones, or a few among small ones) bind the kernel by these atomics, which
// go to the same few lines of memory: one set per wave took 124 us where 8,192
// Gaussians are in the lists of 840 of 1,200 tiles each, one per tile 52 (4 pixels
// per lane, one wave per tile: 49). The waves meet once per span, which costs most
// where few tiles have long lists of small splats (20,000 Gaussians of 2 tiles each
// in 16 tiles: 401 -> 506 us, in 475 tiles 93 -> 95).
template <int kRows>
struct TileSums {
    float v[kRows * kAccStride];
    uint32_t id[kRows];
    uint32_t stop[4];

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < kAccStride; ++i) v[i * kRows + threadIdx.x] = 0.f;
    }
    __device__ __forceinline__ void add(int row, int entry, float x)
    {
        __hip_atomic_fetch_add(&v[row * kAccStride + entry], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // By the whole workgroup: the sums that are not zero into the accumulators of
    // their Gaussians (my_id: the span's entry threadIdx.x), then cleared. Consecutive
    // lanes take consecutive entries of a row.
    __device__ __forceinline__ void flush(uint32_t my_id, float* __restrict__ acc)
    {
        id[threadIdx.x] = my_id;
        __syncthreads();
#pragma unroll 3   // all nine at once take 24 registers more
        for (int i = 0; i < kAccStride; ++i) {
            const int k = i * kRows + (int)threadIdx.x, row = k / kAccStride;
            const float x = v[k];
            v[k] = 0.f;
            if (x != 0.f)
                __hip_atomic_fetch_add(acc + (size_t)id[row] * kAccStride + (k - row * kAccStride), x, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
    }
};

template <>
struct TileSums<0> {};

template <int kPix>
__global__ __launch_bounds__(kTile * kTile / kPix) void k_blend_bwd(Cam cam, const gs_splat* __restrict__ splats,
                                                                    const uint32_t* __restrict__ values,
                                                                    const uint32_t* __restrict__ ranges,
                                                                    const float* __restrict__ final_T,
                                                                    const uint32_t* __restrict__ n_contrib,
                                                                    const float* __restrict__ dL_dimage,
                                                                    const uint32_t* __restrict__ order,
                                                                    float* __restrict__ acc)
{
    constexpr int kRowStep = 4;   // pixel k of a lane lies 4k rows below its first
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    const int tile = order ? (blockIdx.x < (unsigned)n_tiles ? (int)order[blockIdx.x] : n_tiles)
                           : tile_of_block(blockIdx.x, n_tiles);
    if (tile >= n_tiles) return;
    const int lane = __lane_id();
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row_lane = lane & 15;
    const int x = tx * kTile + row_lane;
    const int y0 = ty * kTile + 4 * kPix * wave + (lane >> 4);
    const float px = (float)x + 0.5f;
    const uint32_t start = ranges[2 * tile], len = ranges[2 * tile + 1] - start;
    const int64_t hw = (int64_t)cam.width * cam.height;
    // box of this wave's pixel centres, for the same early skip as the forward
    const float box_cx = (float)(tx * kTile) + 8.f, box_hx = 7.5f;
    const float box_lo = (float)(ty * kTile + 4 * kPix * wave) + 0.5f;
    const float box_hi = box_lo + (float)(4 * kPix - 1);
    const float box_cy = 0.5f * (box_lo + box_hi), box_hy = 0.5f * (box_hi - box_lo);

    // A: the colour behind the current splat, as composited, projected on the
    // pixel's upstream gradient g, the only form of it the gradient needs
    float T[kPix], py[kPix], g0[kPix], g1[kPix], g2[kPix], A[kPix];
    uint32_t last[kPix];
    uint32_t stop = 0;
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        const int y = y0 + kRowStep * k;
        py[k] = (float)y + 0.5f;
        T[k] = 1.f;
        g0[k] = g1[k] = g2[k] = 0.f;
        last[k] = 0;
        if (x < cam.width && y < cam.height) {
            const int64_t pix = (int64_t)y * cam.width + x;
            T[k] = final_T[pix];
            last[k] = min(n_contrib[pix], len);
            g0[k] = dL_dimage[pix];
            g1[k] = dL_dimage[hw + pix];
            g2[k] = dL_dimage[2 * hw + pix];
        }
        A[k] = __fmaf_rn(cam.bg[2], g2[k], __fmaf_rn(cam.bg[1], g1[k], cam.bg[0] * g0[k]));
        stop = max(stop, last[k]);
    }
    // list positions [0, stop) can contribute
    for (int o = 32; o > 0; o >>= 1) stop = max(stop, (uint32_t)__shfl_xor((int)stop, o));
    stop = (uint32_t)__builtin_amdgcn_readfirstlane((int)stop);   // uniform: the walk's control stays scalar
    const int nbatch = (int)((stop + kWave - 1) / kWave);
    // several waves per tile: their sums meet in LDS (TileSums) and the tile issues
    // one set of atomics per splat, for spans of kBatches batches
    constexpr int kWaves = kTile * kTile / kPix / kWave, kBatches = kWaves;
    __shared__ TileSums<(kWaves > 1 ? kBatches * kWave : 0)> sums;
    int spans = 1;
    if constexpr (kWaves > 1) {
        if (lane == 0) sums.stop[wave] = stop;
        sums.clear();
        __syncthreads();
        uint32_t tile_stop = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) tile_stop = max(tile_stop, sums.stop[w]);
        spans = __builtin_amdgcn_readfirstlane((int)((tile_stop + kBatches * kWave - 1) / (kBatches * kWave)));
    } else if (stop == 0) {
        return;
    }
    // each batch of 64 list entries is staged in LDS and read back one record
    // per step at a uniform address (broadcast), as in the forward
    __shared__ StageSlot stage[kTile * kTile / kPix / kWave];
    StageSlot& st = stage[wave];
    // lane roles of the reduction (wave_reduce9)
    const bool red_up = lane & 32, red_hi8 = lane & 8, red_odd4 = lane & 4;
    // A splat's nine sums into its row: of the tile's sums in LDS, from the lanes
    // that hold them; or of the accumulators, gathered into lanes 0..8 by one LDS
    // permute, so that the atomics stay one request per 64 bytes (from four rows of
    // lanes they are four, which at 3M Gaussians costs 0.09 ms).
    const int red_lane = kWaves > 1 ? reduce_entry(lane) : 4 * reduce_src_lane(lane);
    auto add_sums = [&](float u, int span_row, uint32_t batch_id, int j) {
        if constexpr (kWaves > 1) {
            if (red_lane >= 0) sums.add(span_row + j, red_lane, u);
        } else {
            const float t = __int_as_float(__builtin_amdgcn_ds_bpermute(red_lane, __float_as_int(u)));
            const uint32_t id = (uint32_t)__builtin_amdgcn_readlane((int)batch_id, j);
            if (lane < kAccStride) add_scalar_row(acc + (size_t)id * kAccStride, lane, t);
        }
    };
    float4 c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0, c2 = c0;
    uint32_t cid = 0, nid = 0;   // nid: the list entry of the batch after the prefetched one, loaded a batch early
    {
        const uint32_t p = (uint32_t)(nbatch - 1) * kWave + lane;
        if (p < stop) {
            cid = values[start + p];
            const float4* r = reinterpret_cast<const float4*>(splats + cid);
            c0 = r[0]; c1 = r[1]; c2 = r[2];
        }
        if (nbatch >= 2) nid = values[start + (uint32_t)(nbatch - 2) * kWave + lane];
    }
    int bi = nbatch - 1;
    for (int span = spans - 1; span >= 0; --span) {
        // the span's list entries, needed when it is flushed
        [[maybe_unused]] uint32_t span_id = 0;
        if constexpr (kWaves > 1) {
            const uint32_t p = (uint32_t)span * (kBatches * kWave) + threadIdx.x;
            if (p < len) span_id = values[start + p];
        }
        for (; bi >= span * kBatches; --bi) {
            const uint32_t b = (uint32_t)bi * kWave;
            const int span_row = (bi - span * kBatches) * kWave;
            stage_words_bwd(c0, c1, c2, st.w[0][lane], st.w[1][lane], st.w[2][lane]);
            const uint32_t batch_id = cid;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int cnt = (int)min((uint32_t)kWave, stop - b);
            // a splat that reaches alpha >= 1/255 nowhere in this wave's pixels
            // passes nothing back: each lane tests the record it holds (the
            // conservative bounding box, then the ellipse), and the walk visits only
            // the others, back to front
            uint64_t todo = __ballot(lane < cnt && fabsf(c0.x - box_cx) <= c2.z + box_hx &&
                                     fabsf(c0.y - box_cy) <= c2.w + box_hy &&
                                     ellipse_meets_box(c0.x, c0.y, c0.z, c0.w, c1.x, c2.y, box_cx - box_hx,
                                                       box_cx + box_hx, box_lo, box_hi));
            if (bi > 0) {
                cid = nid;
                const float4* r = reinterpret_cast<const float4*>(splats + cid);
                c0 = r[0]; c1 = r[1]; c2 = r[2];
                if (bi > 1) nid = values[start + b - 2 * kWave + lane];
            }
            if constexpr (kPix == 1) {
                // few tiles: kBwdGroup splats a step, without branches, as in the forward;
                // the transmittance and the colour behind go from one to the next. A
                // lane that a splat does not reach takes its values by selects (a
                // product with zero would pass on an infinite colour or gradient).
                while (todo != 0) {
                    StagedBwd s[kBwdGroup];
                    float dx[kBwdGroup], dy[kBwdGroup], oG[kBwdGroup], alpha[kBwdGroup], inv[kBwdGroup];
                    uint64_t in[kBwdGroup];
                    int js[kBwdGroup];
                    int j = 0;
#pragma unroll
                    for (int g = 0; g < kBwdGroup; ++g) {
                        const uint64_t some = todo != 0 ? ~0ull : 0ull;   // none left: the last one again, masked out
                        j = todo != 0 ? 63 - (int)__builtin_clzll(todo) : j;
                        todo &= ~(1ull << j);
                        s[g] = staged_bwd(st.w[0][j], st.w[1][j], st.w[2][j]);
                        js[g] = j;
                        in[g] = some;
                    }
#pragma unroll
                    for (int g = 0; g < kBwdGroup; ++g) {
                        dx[g] = px - s[g].mx;
                        dy[g] = py[0] - s[g].my;
                        const float e = quad_neg_power(s[g], column_quad(s[g], dx[g]), dy[g]);
                        in[g] &= __ballot(b + (uint32_t)js[g] < last[0]) & __ballot(in_reach(e, s[g].e_max));
                        oG[g] = s[g].op * __builtin_amdgcn_exp2f(-e);
                        alpha[g] = __builtin_amdgcn_inverse_ballot_w64(in[g]) ? fminf(kAlphaMax, oG[g]) : 0.f;
                        inv[g] = __builtin_amdgcn_rcpf(1.f - alpha[g]);
                    }
                    float p0[kBwdGroup], p1[kBwdGroup], p2[kBwdGroup], ac0[kBwdGroup], ac1[kBwdGroup], ac2[kBwdGroup];
#pragma unroll
                    for (int g = 0; g < kBwdGroup; ++g) {
                        const bool on = __builtin_amdgcn_inverse_ballot_w64(in[g]);
                        T[0] *= inv[g];
                        const float w = alpha[g] * T[0];
                        ac0[g] = on ? w * g0[0] : 0.f;
                        ac1[g] = on ? w * g1[0] : 0.f;
                        ac2[g] = on ? w * g2[0] : 0.f;
                        const float u =
                            __fmaf_rn(s[g].b, g2[0], __fmaf_rn(s[g].g, g1[0], __fmaf_rn(s[g].r, g0[0], -A[0])));
                        A[0] = on ? __fmaf_rn(alpha[g], u, A[0]) : A[0];
                        p0[g] = on && oG[g] < kAlphaMax ? w * u : 0.f;
                        p1[g] = p0[g] * dy[g];
                        p2[g] = p1[g] * dy[g];
                    }
                    float t[kBwdGroup];
#pragma unroll
                    for (int g = 0; g < kBwdGroup; ++g) {
                        float gx, gy;
                        mean_terms(s[g], dx[g], p0[g], p1[g], gx, gy);
                        t[g] = wave_reduce9(p0[g], p1[g], p2[g], gx, gy, ac0[g], ac1[g], ac2[g], dx[g], red_up, red_hi8,
                                            red_odd4);
                    }
#pragma unroll
                    for (int g = 0; g < kBwdGroup; ++g) {
                        if (in[g] == 0) continue;
                        add_sums(t[g], span_row, batch_id, js[g]);
                    }
                }
            } else {
                while (todo != 0) {
                    const int j = 63 - (int)__builtin_clzll(todo);
                    todo ^= 1ull << j;
                    const uint32_t pos = b + (uint32_t)j;
                    const StagedBwd s = staged_bwd(st.w[0][j], st.w[1][j], st.w[2][j]);
                    const float dx = px - s.mx;
                    const Quad q = column_quad(s, dx);
                    // per-lane sums over its pixels: colour gradient and dL/dpower times
                    // 1, dy, dy^2 (the lane's pixels share dx)
                    float a_c0 = 0.f, a_c1 = 0.f, a_c2 = 0.f;
                    float p0 = 0.f, p1 = 0.f, p2 = 0.f;
                    uint64_t any = 0;
#pragma unroll
                    for (int k = 0; k < kPix; ++k) {
                        // one branch per pixel (no short circuit); the cap is a select inside it
                        const float dy = py[k] - s.my;
                        const float e = quad_neg_power(s, q, dy);
                        // the comparisons' lane masks, combined as scalars
                        const uint64_t reach = __ballot(pos < last[k]) & __ballot(in_reach(e, s.e_max));
                        any |= reach;
                        if (!__builtin_amdgcn_inverse_ballot_w64(reach)) continue;
                        const float oG = s.op * __builtin_amdgcn_exp2f(-e);
                        const float alpha = fminf(kAlphaMax, oG);
                        // hardware reciprocal (1 ulp): T is recovered over a few hundred
                        // splats, so its relative error stays near 1e-5
                        T[k] *= __builtin_amdgcn_rcpf(1.f - alpha);   // transmittance in front of this splat
                        const float w = alpha * T[k];
                        a_c0 = __fmaf_rn(w, g0[k], a_c0);
                        a_c1 = __fmaf_rn(w, g1[k], a_c1);
                        a_c2 = __fmaf_rn(w, g2[k], a_c2);
                        // colour less what it hides, on g: dL/dalpha = T u
                        const float u = __fmaf_rn(s.b, g2[k], __fmaf_rn(s.g, g1[k], __fmaf_rn(s.r, g0[k], -A[k])));
                        A[k] = __fmaf_rn(alpha, u, A[k]);
                        // dL/dpower = alpha dL/dalpha below the cap; a capped entry passes nothing
                        const float dpow = oG < kAlphaMax ? w * u : 0.f;
                        const float pdy = dpow * dy;
                        p0 += dpow;
                        p1 += pdy;
                        p2 = __fmaf_rn(pdy, dy, p2);
                    }
                    if (any == 0) continue;
                    float gx, gy;
                    mean_terms(s, dx, p0, p1, gx, gy);
                    add_sums(wave_reduce9(p0, p1, p2, gx, gy, a_c0, a_c1, a_c2, dx, red_up, red_hi8, red_odd4),
                             span_row, batch_id, j);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        if constexpr (kWaves > 1) sums.flush(span_id, acc);
    }
}

hipError_t launch_blend_bwd(const Cam& cam, const gs_splat* splats, const uint32_t* values,
                            const uint32_t* tile_ranges, const float* final_T, const uint32_t* n_contrib,
                            const float* dL_dimage, const uint32_t* tile_order, float* acc, hipStream_t s)
{
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    auto launch = [&](auto kernel, int pix) {
        hipLaunchKernelGGL(kernel, dim3(tile_order ? n_tiles : blend_grid(n_tiles)), dim3(kTile * kTile / pix), 0, s,
                           cam, splats, values, tile_ranges, final_T, n_contrib, dL_dimage, tile_order, acc);
    };
    switch (bwd_pix(n_tiles)) {
    case 1: launch(k_blend_bwd<1>, 1); break;
    case 2: launch(k_blend_bwd<2>, 2); break;
    default: launch(k_blend_bwd<4>, 4); break;
    }
    return hipGetLastError();
}

// ---- tile order of the backward -----------------------------------------------
// The backward's work in a tile follows the longest walk among its pixels (the
// list up to the last entry any of them blended), and that walk differs by a
// factor of 3 or more between tiles. Workgroups are dispatched in launch order
// and every tile's workgroup is resident at once, so each SIMD gets every
// 1024th tile of the launch order: in list order its share of long walks
// varies, and the SIMD with the most sets the kernel's duration. Launching
// the tiles longest walk first deals each SIMD one tile of every length class.
// The order is taken by a counting sort over 16 classes per octave of the walk
// length; tiles of one class come out in no fixed order (the results do not
// depend on it, beyond the float atomics' summation order).

__device__ __forceinline__ uint32_t walk_class(uint32_t walk)
{
    // exponent and the 4 leading mantissa bits of the walk length as a float:
    // 16 classes per octave, 0 .. kWalkClasses - 1 (walks of 0 and 1 share class 0)
    const uint32_t b = __float_as_uint((float)max(walk, 1u)) >> 19;
    return min(b - (127u << 4), (uint32_t)kWalkClasses - 1);   // 2^32 - 1 rounds up to 2^32
}

// Walk class of each tile, one wave per tile (workgroup `blk` of the walk).
__device__ __forceinline__ void tile_walk(const Cam& cam, const uint32_t* __restrict__ ranges,
                                          const uint32_t* __restrict__ n_contrib, uint32_t* __restrict__ walk_cls,
                                          int blk)
{
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    const int tile = blk * (kBlock / kWave) + (int)(threadIdx.x / kWave);
    if (tile >= n_tiles) return;   // whole waves
    const int lane = __lane_id();
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    const int x = tx * kTile + (lane & 15);
    uint32_t walk = 0;
#pragma unroll
    for (int k = 0; k < kTile / 4; ++k) {
        const int y = ty * kTile + (lane >> 4) + 4 * k;
        if (x < cam.width && y < cam.height) walk = max(walk, n_contrib[(int64_t)y * cam.width + x]);
    }
    for (int o = 32; o > 0; o >>= 1) walk = max(walk, (uint32_t)__shfl_xor((int)walk, o));
    if (lane == 0) walk_cls[tile] = walk_class(min(walk, ranges[2 * tile + 1] - ranges[2 * tile]));
}

// Zeroes p[0, count) as workgroup `blk` of `nblk` (16-byte stores, grid-stride).
__device__ __forceinline__ void clear_part(float* __restrict__ p, int64_t count, int blk, int nblk)
{
    const int64_t c4 = count >> 2;
    const int64_t stride = (int64_t)nblk * kBlock;
    float4* p4 = reinterpret_cast<float4*>(p);
    for (int64_t i = (int64_t)blk * kBlock + threadIdx.x; i < c4; i += stride) p4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (blk == 0 && threadIdx.x < (count & 3)) p[(c4 << 2) + threadIdx.x] = 0.f;
}

// The backward's preparation in one launch: the first walk_blocks workgroups
// take the tiles' walk classes (none when the tiles are not ordered), the
// others clear the screen-space accumulators.
__global__ __launch_bounds__(kBlock) void k_walk_clear(Cam cam, const uint32_t* __restrict__ ranges,
                                                       const uint32_t* __restrict__ n_contrib,
                                                       uint32_t* __restrict__ walk_cls, int walk_blocks,
                                                       float* __restrict__ acc, int64_t count)
{
    const int blk = (int)blockIdx.x;
    if (blk < walk_blocks)
        tile_walk(cam, ranges, n_contrib, walk_cls, blk);
    else
        clear_part(acc, count, blk - walk_blocks, (int)gridDim.x - walk_blocks);
}

constexpr int kOrderThreads = 1024;

__global__ __launch_bounds__(kOrderThreads) void k_tile_order(int n_tiles, const uint32_t* __restrict__ walk_cls,
                                                              uint32_t* __restrict__ order)
{
    __shared__ uint32_t cnt[kWalkClasses];
    __shared__ uint32_t scan[2][kWalkClasses];
    const int t = threadIdx.x;
    for (int c = t; c < kWalkClasses; c += kOrderThreads) cnt[c] = 0;
    __syncthreads();
    for (int i = t; i < n_tiles; i += kOrderThreads) atomicAdd(&cnt[walk_cls[i]], 1u);
    __syncthreads();
    // first position of each class, the longest class first: the sum of the
    // counts of all longer classes (inclusive scan over the reversed classes)
    int src = 0;
    for (int c = t; c < kWalkClasses; c += kOrderThreads) scan[0][c] = cnt[kWalkClasses - 1 - c];
    __syncthreads();
    for (int d = 1; d < kWalkClasses; d <<= 1) {
        for (int c = t; c < kWalkClasses; c += kOrderThreads)
            scan[src ^ 1][c] = scan[src][c] + (c >= d ? scan[src][c - d] : 0u);
        __syncthreads();
        src ^= 1;
    }
    for (int c = t; c < kWalkClasses; c += kOrderThreads) {
        const int r = kWalkClasses - 1 - c;   // reversed index of class c
        cnt[c] = scan[src][r] - cnt[c];       // counts of the classes above c
    }
    __syncthreads();
    for (int i = t; i < n_tiles; i += kOrderThreads) order[atomicAdd(&cnt[walk_cls[i]], 1u)] = (uint32_t)i;
}

// Images of no more tiles than compute units gain nothing from an order (64
// tiles: 9.2 us of preparation and 76 of backward with it, 6.4 and 75 without;
// 300 tiles 9.6 + 98 and 6.7 + 97, but 600 tiles 9.9 + 90 and 6.6 + 115).
bool tile_order_wanted(const Cam& cam)
{
    const int64_t tiles = (int64_t)cam.tiles_x * cam.tiles_y;
    return tiles > kMinOrderedTiles && tiles <= kMaxOrderedTiles;
}

hipError_t launch_bwd_prep(const Cam& cam, const uint32_t* tile_ranges, const uint32_t* n_contrib, float* acc,
                           int64_t acc_count, uint32_t* walk_cls, uint32_t* order, hipStream_t s)
{
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    const int walk_blocks = order ? (int)div_up(n_tiles, kBlock / kWave) : 0;
    const int clear_blocks = (int)std::min<int64_t>(std::max<int64_t>(div_up(acc_count >> 2, kBlock), 1), 4096);
    hipLaunchKernelGGL(k_walk_clear, dim3((unsigned)(walk_blocks + clear_blocks)), dim3(kBlock), 0, s, cam,
                       tile_ranges, n_contrib, walk_cls, walk_blocks, acc, acc_count);
    if (order) hipLaunchKernelGGL(k_tile_order, dim3(1), dim3(kOrderThreads), 0, s, n_tiles, walk_cls, order);
    return hipGetLastError();
}

// ---- work counts (measurement) ------------------------------------------------
// Walks every pixel's list with the forward's decisions (the same fp32
// operations as k_blend_fwd) and counts, per pixel: entries blended; entries
// evaluated in the forward (up to the stop entry, or the list's end, whose
// alpha >= 1/255 box meets the tile: the blend kernels skip the others for
// the whole tile without a per-pixel test); evaluated entries before the last
// blended one (those the backward evaluates); that last position
// (n_contrib); and the entries the method visits in the forward (up to and
// including the stop entry, or the whole list). One wave per tile, 4 pixels
// per lane; per-wave sums, then one 64-bit atomic per wave and counter.
__global__ __launch_bounds__(kWave) void k_blend_count(Cam cam, const gs_splat* __restrict__ splats,
                                                       const uint32_t* __restrict__ values,
                                                       const uint32_t* __restrict__ ranges,
                                                       unsigned long long* __restrict__ counts)
{
    constexpr int kPix = 4, kRowStep = 4;
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    const int tile = blockIdx.x;
    if (tile >= n_tiles) return;
    const int lane = __lane_id();
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    const int x = tx * kTile + (lane & 15);
    const int y0 = ty * kTile + (lane >> 4);
    const float px = (float)x + 0.5f;
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
    const float box_cx = (float)(tx * kTile) + 8.f, box_hx = 7.5f;
    const float box_cy = (float)(ty * kTile) + 8.f, box_hy = 7.5f;
    float T[kPix], py[kPix];
    uint32_t blended[kPix], eval_fwd[kPix], eval_bwd[kPix], pending[kPix], last[kPix], walked[kPix];
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        py[k] = (float)(y0 + kRowStep * k) + 0.5f;
        T[k] = (x < cam.width && (y0 + kRowStep * k) < cam.height) ? 1.f : -1.f;
        blended[k] = eval_fwd[k] = eval_bwd[k] = pending[k] = last[k] = walked[k] = 0;
    }
    for (uint32_t p = start; p < end; ++p) {
#pragma unroll
        for (int k = 0; k < kPix; ++k) walked[k] += T[k] > 0.f ? 1u : 0u;   // visited while blending
        const float4* rec = reinterpret_cast<const float4*>(splats + values[p]);
        const float4 c0 = rec[0], c1 = rec[1], c2 = rec[2];
        if (!(fabsf(c0.x - box_cx) <= c2.z + box_hx && fabsf(c0.y - box_cy) <= c2.w + box_hy)) continue;
        float4 w0, w1;
        float2 w2;
        stage_words(c0, c1, c2, w0, w1, w2);
        const Staged s = staged(w0, w1, w2);
        const float dx = px - s.mx;
        const Quad q = column_quad(s, dx);
#pragma unroll
        for (int k = 0; k < kPix; ++k) {
            if (!(T[k] > 0.f)) continue;
            ++eval_fwd[k];
            const float e = quad_neg_power(s, q, py[k] - s.my);
            if (!in_reach(e, s.e_max)) { ++pending[k]; continue; }
            const float alpha = fminf(kAlphaMax, s.op * __builtin_amdgcn_exp2f(-e));
            const float Tn = T[k] * (1.f - alpha);
            if (Tn < kTMin) { T[k] = -T[k]; continue; }
            T[k] = Tn;
            ++blended[k];
            eval_bwd[k] += pending[k] + 1;
            pending[k] = 0;
            last[k] = p - start + 1;
        }
    }
    unsigned long long c[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        if (x >= cam.width || y0 + kRowStep * k >= cam.height) continue;
        c[0] += blended[k];
        c[1] += last[k];
        c[2] += eval_bwd[k];
        c[3] += eval_fwd[k];
        c[4] += walked[k];
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        unsigned long long v = c[i];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) atomicAdd(counts + i, v);
    }
}

hipError_t launch_blend_count(const Cam& cam, const gs_splat* splats, const uint32_t* values,
                              const uint32_t* tile_ranges, uint64_t* counts, hipStream_t s)
{
    hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t*>(counts), 10, 0u, s);
    if (e != hipSuccess) return e;
    const int n_tiles = cam.tiles_x * cam.tiles_y;
    hipLaunchKernelGGL(k_blend_count, dim3(n_tiles), dim3(kWave), 0, s, cam, splats, values, tile_ranges,
                       reinterpret_cast<unsigned long long*>(counts));
    return hipGetLastError();
}

// Zero fill of `count` floats; p must be 16-byte aligned. Body in float4, tail
// in scalars. A kernel rather than a memset so that it behaves the same inside
// a captured graph.
__global__ __launch_bounds__(kBlock) void k_clear(float* __restrict__ p, int64_t count)
{
    clear_part(p, count, (int)blockIdx.x, (int)gridDim.x);
}

hipError_t launch_clear(float* p, int64_t count, hipStream_t s)
{
    const int blocks = (int)std::min<int64_t>(std::max<int64_t>(div_up(count >> 2, kBlock), 1), 4096);
    hipLaunchKernelGGL(k_clear, dim3(blocks), dim3(kBlock), 0, s, p, count);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t* __restrict__ p, int64_t count, uint32_t v)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += stride) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, int64_t count, uint32_t value, hipStream_t s)
{
    const int blocks = (int)std::min<int64_t>(std::max<int64_t>(div_up(count, kBlock), 1), 4096);
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks), dim3(kBlock), 0, s, p, count, value);
    return hipGetLastError();
}

}  // namespace gsr
