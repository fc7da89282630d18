// thin_kernels.hip -- gfx950 kernels of the lambda-leveling loop and the
// lambda-skeleton.
//
// A parity step t lowers, all at once, the lambda-destructible pixels of the
// parity class s = t mod 4 (classes (i mod 2, j mod 2) = (0,0), (0,1), (1,0),
// (1,1)).  Pixels of one class are never 8-adjacent, so their decisions read
// only pixels no other candidate of the step writes; the result equals
// lowering the class pixel by pixel.
//
// Characterisation of a candidate x with value v (section 2.1):
//   U = {ring neighbours >= v} (Gamma+), L = ring minus U (Gamma--);
//   destructible <=> T+ = #C_n[x, U] = 1 and T-- = #C_n'[x, L] = 1 (a table
//   lookup on the 8-bit mask U);
//   otherwise, when T-- = k >= 2 and lambda > 0, x is lambda-destructible if at
//   least k-1 counted lower components c have v - max_c F <= lambda, i.e.
//   contain a pixel y with v - F(y) <= lambda;
//   a lambda-destructible x gets F(x) := alpha- = max F over L.
// The lambda-skeleton (section 2.2's algorithm box) lowers instead the
// lambda-deletable points that are not lambda-end points: a peak (T+ = 0) is
// lowered too when v - alpha- <= lambda, and an end point (one upper
// n-neighbour) is kept when v - alpha- > lambda.  Its tables carry the peak
// and end bits; the images' table index selects the operator.
//
// Kernels:
//   k_step   one parity step per launch, straight from global memory;
//   k_round  one round: LDS tiles with a halo of K pixels, one residency
//            running K parity steps (the exact region shrinks by one pixel
//            per step), reading one ping-pong buffer and writing the other.
//            A tile whose 3x3 tile neighbourhood lowered nothing during the
//            last 4 steps cannot lower anything in the coming K steps
//            (K <= tile side: every pixel it could read was already examined
//            at the same values), so it is skipped; it only copies itself
//            across the ping-pong pair when it changed during the previous
//            round.  Residency variants (Tile, RTile, BTile) differ only in
//            how a step finds and examines its candidates;
//   k_coop   the rounds of k_round in one cooperative launch;
//   k_flow   small images in one launch: every tile resident from its first
//            step to its last, halos exchanged between running blocks;
//   k_worklist  one block per image, device-side pixel work lists.
#include "thin_internal.h"

#include <climits>
#include <type_traits>

#include <hip/hip_cooperative_groups.h>

namespace thin {

namespace {

constexpr int kThreads = 256;
// Compiled shapes of k_flow: tile height, width, steps between exchanges (the
// halo), threads.
#define THIN_FLOW_SHAPES(X) \
    X(16, 16, 8, 256)       \
    X(24, 48, 8, 640)       \
    X(48, 48, 8, 1024)      \
    X(128, 48, 8, 768)      \
    X(176, 48, 8, 1024)

constexpr int STAGE_CHUNK = 8;  // global loads in flight per thread while staging a tile

// ---------------------------------------------------------------- decision
//
// The decision is VALU-bound wherever whole waves examine candidates, so it
// works on the ring in pairs: four registers of two 16-bit neighbours, one
// with the centre twice.  d = saturating centre - neighbour is nonzero
// exactly for the lower neighbours (L), d - lambda for those out of lambda's
// reach, and the least d - 1 over L (a zero d wraps to the top) is the
// contrast less one.  Each mask costs a packed minimum with 1, three
// shift-ors and one dot product that places both halves.

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u16x2 as_pair(uint32_t x) { return __builtin_bit_cast(u16x2, x); }
__device__ __forceinline__ uint32_t as_word(u16x2 x) { return __builtin_bit_cast(uint32_t, x); }

// (1, 1), hidden from the optimiser: it would turn the packed minimum with a
// known 1 into two compares and selects.
__device__ __forceinline__ u16x2 pair_of_ones()
{
    uint32_t one = 0x00010001u;
    asm("" : "+s"(one));
    return as_pair(one);
}

// lambda as the decision takes it: contrasts are at most 65535.
struct Lambda {
    uint32_t one;   // min(lambda, 65535)
    u16x2 two;      // the same in both halves
};
__device__ __forceinline__ Lambda lambda_of(uint32_t lambda)
{
    Lambda l;
    l.one = lambda < 65535u ? lambda : 65535u;
    l.two = as_pair(l.one * 0x00010001u);
    return l;
}

// The ring around a candidate: p0 = (NW, N), p1 = (SW, S), p2 = (NE, SE),
// p3 = (W, E), first in the low half; v = the candidate in both halves.
struct Ring {
    u16x2 p0, p1, p2, p3, v;
};

// From the 16-bit neighbours E, NE, N, NW, W, SW, S, SE.
__device__ __forceinline__ Ring ring_of(uint32_t v, const uint32_t (&nb)[8])
{
    return Ring{as_pair(nb[3] | nb[2] << 16), as_pair(nb[5] | nb[6] << 16),
                as_pair(nb[1] | nb[7] << 16), as_pair(nb[4] | nb[0] << 16),
                as_pair(v * 0x00010001u)};
}

// From three rows of bytes (W, centre, E in the low three bytes).
__device__ __forceinline__ Ring ring_of_bytes(uint32_t up, uint32_t mid, uint32_t down)
{
    return Ring{as_pair(__builtin_amdgcn_perm(0u, up, 0x0C010C00u)),
                as_pair(__builtin_amdgcn_perm(0u, down, 0x0C010C00u)),
                as_pair(__builtin_amdgcn_perm(down, up, 0x0C060C02u)),
                as_pair(__builtin_amdgcn_perm(0u, mid, 0x0C020C00u)),
                as_pair(__builtin_amdgcn_perm(0u, mid, 0x0C010C01u))};
}

// From three rows of four 16-bit pixels (two words each), the candidate in
// column 1 (RIGHT = false) or 2 (RIGHT = true).
template <bool RIGHT>
__device__ __forceinline__ Ring ring_of_words(uint32_t u0, uint32_t u1, uint32_t m0, uint32_t m1,
                                              uint32_t d0, uint32_t d1)
{
    constexpr uint32_t straddle = 0x05040302u;  // high half of word 0, low half of word 1
    if constexpr (!RIGHT)
        return Ring{as_pair(u0), as_pair(d0), as_pair(__builtin_amdgcn_perm(d1, u1, 0x05040100u)),
                    as_pair(__builtin_amdgcn_perm(m1, m0, 0x05040100u)),
                    as_pair(__builtin_amdgcn_perm(0u, m0, 0x03020302u))};
    else
        return Ring{as_pair(__builtin_amdgcn_perm(u1, u0, straddle)),
                    as_pair(__builtin_amdgcn_perm(d1, d0, straddle)),
                    as_pair(__builtin_amdgcn_perm(d1, u1, 0x07060302u)),
                    as_pair(__builtin_amdgcn_perm(m1, m0, 0x07060302u)),
                    as_pair(__builtin_amdgcn_perm(0u, m1, 0x01000100u))};
}

// (x of p0..p3 in the low halves, then in the high halves) as a byte, times scale.
__device__ __forceinline__ uint32_t mask_of(u16x2 b0, u16x2 b1, u16x2 b2, u16x2 b3,
                                            unsigned short scale)
{
    const uint32_t m = (as_word(b0) | as_word(b1) << 1) | (as_word(b2) | as_word(b3) << 1) << 2;
    const u16x2 w = {scale, (unsigned short)(16 * scale)};
    return __builtin_amdgcn_udot2(as_pair(m), w, 0u, false);
}

// A candidate's test in numbers (see DecEntry): it is lowered to alpha (its
// alpha-) when near >= need and, where its own contrast must be within lambda,
// contrast1 < reach.  lut points at the 256 entries of the image's adjacency
// and operator.
struct Verdict {
    uint32_t near, need;        // counted components within lambda's reach: present, needed
    int32_t own;                // negative: its own contrast must be within lambda too
    uint32_t contrast1, reach;  // v - alpha- - 1, and its bound (lambda); or
                                // both subtracted from 65535, the other way round
    uint32_t alpha;

    __device__ __forceinline__ bool lower() const
    {
        return near >= need && (own >= 0 || contrast1 < reach);
    }
    // The wave's lanes that lower (whole-wave compares and scalar logic: asked
    // for lower() in one ballot the compiler goes through a register of 0 and 1).
    __device__ __forceinline__ uint64_t lanes() const
    {
        return __ballot(near >= need) & (__ballot(own >= 0) | __ballot(contrast1 < reach));
    }
};
// How many of the components hold a pixel that is not in far.
__device__ __forceinline__ uint32_t components_near(uint32_t comps, uint32_t far)
{
    const uint32_t hit = comps & ~__builtin_amdgcn_perm(0u, far, 0u);
    return (uint32_t)__popc((((hit & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | hit) & 0x80808080u);
}
__device__ __forceinline__ Verdict weigh(const Ring& q, const DecEntry* lut, const Lambda& lam)
{
    const u16x2 one = pair_of_ones();
    const u16x2 d0 = __builtin_elementwise_sub_sat(q.v, q.p0);
    const u16x2 d1 = __builtin_elementwise_sub_sat(q.v, q.p1);
    const u16x2 d2 = __builtin_elementwise_sub_sat(q.v, q.p2);
    const u16x2 d3 = __builtin_elementwise_sub_sat(q.v, q.p3);
    const uint32_t at = mask_of(__builtin_elementwise_min(d0, one), __builtin_elementwise_min(d1, one),
                                __builtin_elementwise_min(d2, one), __builtin_elementwise_min(d3, one),
                                sizeof(DecEntry));
    const uint64_t raw = *reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(lut) + at);
    const uint32_t need = (uint32_t)raw, comps = (uint32_t)(raw >> 32);
    auto beyond = [&](u16x2 d) __attribute__((always_inline)) {
        return __builtin_elementwise_min(__builtin_elementwise_sub_sat(d, lam.two), one);
    };
    const uint32_t far = mask_of(beyond(d0), beyond(d1), beyond(d2), beyond(d3), 1);
    const u16x2 c = __builtin_elementwise_min(__builtin_elementwise_min(d0 - one, d1 - one),
                                              __builtin_elementwise_min(d2 - one, d3 - one));
    Verdict v;
    v.near = components_near(comps, far);
    v.need = need & 0xFFu;
    v.contrast1 = min(as_word(c) & 0xFFFFu, as_word(c) >> 16);
    v.reach = lam.one;
    v.own = (int32_t)need;
    v.alpha = (as_word(q.v) & 0xFFFFu) - 1u - v.contrast1;
    return v;
}
// The same for pixels and lambda of at most 255.  The differences fit 16 bits
// with their sign, so one subtraction a pair serves all: its signs are L, the
// signs after adding lambda the pixels out of reach, and its largest value as
// an unsigned number is that of the highest lower neighbour.  A permute turns
// four signs into bytes of 0 or -1, and dot products with the negative powers
// of two make a mask of them: 32 instructions where weigh() takes 43.  Only the
// bit-flag tiles hold one pixel type a kernel; the register windows, whose
// steps are chains of latencies, decide both types by weigh().
__device__ __forceinline__ Verdict weigh_small(const Ring& q, const DecEntry* lut, const Lambda& lam)
{
    const u16x2 x0 = q.p0 - q.v, x1 = q.p1 - q.v, x2 = q.p2 - q.v, x3 = q.p3 - q.v;
    auto signs = [](u16x2 a, u16x2 b, u16x2 c, u16x2 d) __attribute__((always_inline)) {
        constexpr uint32_t of_halves = 0x0B0A0908u;  // the sign of each half of both operands
        const int ab = (int)__builtin_amdgcn_perm(as_word(b), as_word(a), of_halves);
        const int cd = (int)__builtin_amdgcn_perm(as_word(d), as_word(c), of_halves);
        // -1 times -1, -16, -2, -32 and -4, -64, -8, -128
        return (uint32_t)__builtin_amdgcn_sdot4(
            cd, (int)0x80F8C0FCu, __builtin_amdgcn_sdot4(ab, (int)0xE0FEF0FFu, 0, false), false);
    };
    const uint32_t at = signs(x0, x1, x2, x3) * (uint32_t)sizeof(DecEntry);
    const uint64_t raw = *reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(lut) + at);
    const uint32_t need = (uint32_t)raw, comps = (uint32_t)(raw >> 32);
    const u16x2 top2 = __builtin_elementwise_max(__builtin_elementwise_max(x0, x1),
                                                 __builtin_elementwise_max(x2, x3));
    const uint32_t top = max(as_word(top2) & 0xFFFFu, as_word(top2) >> 16);
    Verdict v;
    v.near = components_near(comps, signs(x0 + lam.two, x1 + lam.two, x2 + lam.two, x3 + lam.two));
    v.need = need & 0xFFu;
    v.own = (int32_t)need;
    v.contrast1 = 0xFFFFu - lam.one;
    v.reach = top;
    v.alpha = ((as_word(q.v) & 0xFFFFu) + top) & 0xFFFFu;
    return v;
}
__device__ __forceinline__ bool decide(const Ring& q, const DecEntry* lut, const Lambda& lam,
                                       uint32_t& alpha)
{
    const Verdict v = weigh(q, lut, lam);
    alpha = v.alpha;
    return v.lower();
}

__device__ __forceinline__ uint32_t load_px(const void* base, int dtype, int64_t idx)
{
    return dtype == 1 ? (uint32_t)static_cast<const uint8_t*>(base)[idx]
                      : (uint32_t)static_cast<const uint16_t*>(base)[idx];
}

__device__ __forceinline__ void store_px(void* base, int dtype, int64_t idx, uint32_t v)
{
    if (dtype == 1) static_cast<uint8_t*>(base)[idx] = (uint8_t)v;
    else static_cast<uint16_t*>(base)[idx] = (uint16_t)v;
}

// ------------------------------------------------------------------ k_init

__global__ void k_init_state(ImgCnt* cnt, int nimg, int32_t* tile_last, int ntiles,
                             int32_t* hist_round, WorkList wl)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (wl.list != nullptr) {
        if (i < ntiles) wl.listed[i] = -1;
        if (i < 3) wl.count[i] = 0;
        if (i < 6) wl.grab[i] = 0;
    }
    if (hist_round && i < 2 * ntiles) hist_round[i] = -1;
    if (i < nimg) {
        cnt[i].lowerings = 0ull;
        cnt[i].tile_rounds = 0ull;
        cnt[i].last_step = -1;
        cnt[i].pad = -1;
        cnt[i].examinations = 0ull;
    }
    if (tile_last && i < 2 * ntiles) tile_last[i] = -1;
}

// One block per image.
__global__ void k_serve_init(const ImgDev* __restrict__ imgs, ImgCnt* cnt, int32_t* tile_state)
{
    const ImgDev* d = imgs + blockIdx.x;
    if (d->fresh == 0) return;
    if (threadIdx.x == 0) {
        ImgCnt* c = cnt + d->slot;
        c->lowerings = 0ull;
        c->tile_rounds = 0ull;
        c->last_step = -1;
        c->pad = -1;
        c->examinations = 0ull;
    }
    const int n = 2 * d->tiles_x * d->tiles_y;
    for (int i = threadIdx.x; i < n; i += blockDim.x) tile_state[2 * d->state0 + i] = -1;
}

__global__ void k_set_desc(ImgDev* dst, ImgDev d)
{
    if (threadIdx.x == 0) *dst = d;
}

__global__ void k_advance(int32_t* round_base, int n)
{
    if (threadIdx.x == 0) *round_base += n;
}

// ------------------------------------------------------------------ k_step

template <typename T>
__global__ __launch_bounds__(kThreads) void k_step(const ImgDev* __restrict__ img, ImgCnt* cnt,
                                                   int step, const DecEntry* __restrict__ lut_g)
{
    __shared__ DecEntry s_lut[256];
    const ImgDev d = *img;
    for (int i = threadIdx.x; i < 256; i += kThreads) s_lut[i] = lut_g[d.adj * 256 + i];
    __syncthreads();
    const int s = step & 3, si = s >> 1, sj = s & 1;
    const int i = 2 * (int)blockIdx.y + si;
    const int j = 2 * (int)(blockIdx.x * kThreads + threadIdx.x) + sj;
    bool lowered = false;
    const bool inside = i >= 1 && i <= d.h - 2 && j >= 1 && j <= d.w - 2;
    if (inside) {
        T* px = static_cast<T*>(d.buf[0]) + (int64_t)i * d.pitch + j;
        const int64_t P = d.pitch;
        const uint32_t v = px[0];
        const uint32_t nb[8] = {px[1], px[-P + 1], px[-P], px[-P - 1],
                                px[-1], px[P - 1], px[P], px[P + 1]};
        uint32_t alpha;
        if (decide(ring_of(v, nb), s_lut, lambda_of(d.lambda), alpha)) {
            px[0] = (T)alpha;
            lowered = true;
        }
    }
    const unsigned long long ballot = __ballot(lowered);
    const unsigned long long seen = __ballot(inside);
    if ((threadIdx.x & 63) == 0 && seen != 0ull)
        atomicAdd(&cnt->examinations, (unsigned long long)__popcll(seen));
    if ((threadIdx.x & 63) == 0 && ballot != 0ull) {
        atomicAdd(&cnt->lowerings, (unsigned long long)__popcll(ballot));
        atomicMax(&cnt->last_step, step);
    }
}

// ------------------------------------------------------------ tile residency

// Scalar fields of an image used inside a residency (no arrays, so the
// compiler keeps them in registers).
struct View {
    int64_t pitch;
    int32_t h, w;
    int32_t dtype;
    uint32_t lambda;
};

__device__ __forceinline__ View view_of(const ImgDev* d)
{
    View v;
    v.pitch = d->pitch;
    v.h = d->h;
    v.w = d->w;
    v.dtype = d->dtype;
    v.lambda = d->lambda;
    return v;
}

// Ping-pong buffer read by round r (src) and written by it (dst).  The
// descriptor stays in global memory: copying it into a local and indexing its
// array by r & 1 would push the copy into scratch.
__device__ __forceinline__ const void* round_src(const ImgDev* d, int r)
{
    return d->buf[r & 1];
}

__device__ __forceinline__ void* round_dst(const ImgDev* d, int r)
{
    return d->buf[(r + 1) & 1];
}

// ------------------------------------------------------- wide tile transfers
//
// Groups of 4 pixels move as one dword (u8) or two (u16) when both
// ping-pong buffers and the pitch are aligned to a group (the twin is
// 256-byte aligned, so the caller's buffer and pitch decide).  Region and
// interior columns start at multiples of 4, so a group lies wholly left of
// the image or starts inside it; only the last group of a row can be cut by
// the right border, and it moves pixel by pixel.

__device__ __forceinline__ bool wide_ok(const View& d, const void* a, const void* b)
{
    const uintptr_t al = d.dtype == 1 ? 4u : 8u;
    return (d.pitch & 3) == 0 && ((uintptr_t)a % al) == 0 && ((uintptr_t)b % al) == 0;
}

// 4 pixels as two u16 pairs (pixel 0 in the low half of .x).
__device__ __forceinline__ uint2 load4(const uint8_t* p)
{
    const uint32_t w = *reinterpret_cast<const uint32_t*>(p);
    return make_uint2((w & 0xFFu) | ((w << 8) & 0xFF0000u), ((w >> 16) & 0xFFu) | ((w >> 8) & 0xFF0000u));
}
__device__ __forceinline__ uint2 load4(const uint16_t* p) { return *reinterpret_cast<const uint2*>(p); }

__device__ __forceinline__ void store4(uint8_t* p, uint2 v)
{
    *reinterpret_cast<uint32_t*>(p) = (v.x & 0xFFu) | ((v.x >> 8) & 0xFF00u) | ((v.y & 0xFFu) << 16) |
                                      ((v.y << 8) & 0xFF000000u);
}
__device__ __forceinline__ void store4(uint16_t* p, uint2 v) { *reinterpret_cast<uint2*>(p) = v; }

template <typename P>
__device__ __forceinline__ uint2 load_partial(const P* p, int n)
{
    uint32_t q[4] = {0u, 0u, 0u, 0u};
    for (int i = 0; i < n; ++i) q[i] = p[i];
    return make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
}

template <typename P>
__device__ __forceinline__ void store_partial(P* p, uint2 v, int n)
{
    const uint32_t q[4] = {v.x & 0xFFFFu, v.x >> 16, v.y & 0xFFFFu, v.y >> 16};
    for (int i = 0; i < n; ++i) p[i] = (P)q[i];
}

// Region rows [0, RH) x columns [0, RW) of src, origin (ry0, rx0), into
// s_img (u16, row pitch RWP) at (y + OFF, x + OFF), OFF 0 or 1; zeros outside
// the image.
template <typename P, int RH, int RW, int RWP, int OFF, int NT>
__device__ __forceinline__ void stage_wide(const View& d, const P* src, int ry0, int rx0,
                                           uint16_t* s_img, int tid)
{
    static_assert(RW % 4 == 0 && RWP % (OFF ? 2 : 4) == 0 && OFF <= 1, "groups of 4 pixels");
    constexpr int GW = RW / 4, NG = RH * GW;
    constexpr int ITER = (NG + NT - 1) / NT;
    constexpr int CH = ITER < STAGE_CHUNK ? ITER : STAGE_CHUNK;
#pragma unroll 1
    for (int k0 = 0; k0 < ITER; k0 += CH) {
        uint2 v[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int g = tid + (k0 + c) * NT;
            const int y = g / GW, x = 4 * (g - (g / GW) * GW);
            const int gi = ry0 + y, gj = rx0 + x;
            v[c] = make_uint2(0u, 0u);
            if (g < NG && gi >= 0 && gi < d.h && gj >= 0 && gj < d.w) {
                const P* row = src + (int64_t)gi * d.pitch + gj;
                v[c] = gj + 4 <= d.w ? load4(row) : load_partial(row, d.w - gj);
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int g = tid + (k0 + c) * NT;
            if (g < NG) {
                const int y = g / GW, x = 4 * (g - (g / GW) * GW);
                uint16_t* p = s_img + (y + OFF) * RWP + x + OFF;
                if constexpr (OFF == 0) {
                    *reinterpret_cast<uint2*>(p) = v[c];
                } else {  // p + 1 is at a word
                    p[0] = (uint16_t)v[c].x;
                    *reinterpret_cast<uint32_t*>(p + 1) = __builtin_amdgcn_alignbyte(v[c].y, v[c].x, 2);
                    p[3] = (uint16_t)(v[c].y >> 16);
                }
            }
        }
    }
}

// Interior rows [0, TH) x columns [0, TW) of s_img (origin (OY, OX) in it)
// to dst at (gy0, gx0), clipped to the image.
template <typename P, int TH, int TW, int RWP, int OY, int OX, int NT>
__device__ __forceinline__ void store_wide(const View& d, P* dst, int gy0, int gx0,
                                           const uint16_t* s_img, int tid)
{
    static_assert(TW % 4 == 0 && OX % 4 == 0 && RWP % 4 == 0, "groups of 4 pixels");
    constexpr int GW = TW / 4;
    const int ih = min(TH, d.h - gy0), iw = min(TW, d.w - gx0);
    for (int g = tid; g < TH * GW; g += NT) {
        const int y = g / GW, x = 4 * (g - (g / GW) * GW);
        if (y < ih && x < iw) {
            const uint2 v = *reinterpret_cast<const uint2*>(s_img + (OY + y) * RWP + OX + x);
            P* q = dst + (int64_t)(gy0 + y) * d.pitch + gx0 + x;
            if (x + 4 <= iw) store4(q, v);
            else store_partial(q, v, iw - x);
        }
    }
}

// Region rows [0, RH) x columns [0, RW) of src, origin (ry0, rx0), into
// s_img at (y + OY, x + OX) with row pitch RWP, one pixel per load, up to
// STAGE_CHUNK loads in flight per thread (more would cost registers that
// the steps need); zeros outside the image.
template <int RH, int RW, int RWP, int OY, int OX, int NT>
__device__ __forceinline__ void stage_scalar(const View& d, const void* src, int ry0, int rx0,
                                             uint16_t* s_img, int tid)
{
    constexpr int ITER = (RH * RW + NT - 1) / NT;
    constexpr int CH = ITER < STAGE_CHUNK ? ITER : STAGE_CHUNK;
#pragma unroll 1
    for (int k0 = 0; k0 < ITER; k0 += CH) {
        uint32_t vals[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int idx = tid + (k0 + c) * NT;
            const int y = idx / RW, x = idx - y * RW;
            const int gi = ry0 + y, gj = rx0 + x;
            vals[c] = 0;
            if (idx < RH * RW && gi >= 0 && gi < d.h && gj >= 0 && gj < d.w)
                vals[c] = load_px(src, d.dtype, (int64_t)gi * d.pitch + gj);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int idx = tid + (k0 + c) * NT;
            const int y = idx / RW, x = idx - y * RW;
            if (idx < RH * RW) s_img[(y + OY) * RWP + x + OX] = (uint16_t)vals[c];
        }
    }
}

// Staging with groups of 4 pixels where the buffers allow it.
template <int RH, int RW, int RWP, int OFF, int NT>
__device__ __forceinline__ void stage_region(const View& d, const void* src, const void* dst,
                                             int ry0, int rx0, uint16_t* s_img, int tid)
{
    if (wide_ok(d, src, dst)) {
        if (d.dtype == 1)
            stage_wide<uint8_t, RH, RW, RWP, OFF, NT>(d, static_cast<const uint8_t*>(src), ry0, rx0,
                                                      s_img, tid);
        else
            stage_wide<uint16_t, RH, RW, RWP, OFF, NT>(d, static_cast<const uint16_t*>(src), ry0,
                                                       rx0, s_img, tid);
    } else {
        stage_scalar<RH, RW, RWP, OFF, OFF, NT>(d, src, ry0, rx0, s_img, tid);
    }
}

// Interior of the staged region (origin (OY, OX) in s_img) to dst.
template <int TH, int TW, int RWP, int OY, int OX, int NT>
__device__ __forceinline__ void store_region(const View& d, const void* src, void* dst, int gy0,
                                             int gx0, const uint16_t* s_img, int tid)
{
    if constexpr (OX % 4 == 0 && RWP % 4 == 0 && TW % 4 == 0) {
        if (wide_ok(d, src, dst)) {
            if (d.dtype == 1)
                store_wide<uint8_t, TH, TW, RWP, OY, OX, NT>(d, static_cast<uint8_t*>(dst), gy0,
                                                             gx0, s_img, tid);
            else
                store_wide<uint16_t, TH, TW, RWP, OY, OX, NT>(d, static_cast<uint16_t*>(dst), gy0,
                                                              gx0, s_img, tid);
            return;
        }
    }
    const int ih = min(TH, d.h - gy0), iw = min(TW, d.w - gx0);
    for (int idx = tid; idx < TH * TW; idx += NT) {
        const int y = idx / TW, x = idx - y * TW;
        if (y < ih && x < iw)
            store_px(dst, d.dtype, (int64_t)(gy0 + y) * d.pitch + (gx0 + x),
                     s_img[(OY + y) * RWP + (OX + x)]);
    }
}

// Staging and store with the LDS tile in the image's own pixel type E (u8
// tiles take half the LDS of u16 ones).  Groups of 4 pixels move unchanged
// between global memory and LDS where the buffers allow it.
template <typename E>
__device__ __forceinline__ void copy4(E* dst, const E* src)
{
    if constexpr (sizeof(E) == 1) *reinterpret_cast<uint32_t*>(dst) = *reinterpret_cast<const uint32_t*>(src);
    else *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(src);
}

template <typename E, int RH, int RW, int RWP, int NT>
__device__ __forceinline__ void stage_native(const View& d, const void* srcv, const void* dstv,
                                             int ry0, int rx0, E* s_img, int tid)
{
    static_assert(RW % 4 == 0 && RWP % 4 == 0, "groups of 4 pixels");
    const E* src = static_cast<const E*>(srcv);
    if (!wide_ok(d, srcv, dstv)) {
        constexpr int ITER = (RH * RW + NT - 1) / NT;
        constexpr int CH = ITER < STAGE_CHUNK ? ITER : STAGE_CHUNK;
#pragma unroll 1
        for (int k0 = 0; k0 < ITER; k0 += CH) {
            E vals[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int idx = tid + (k0 + c) * NT;
                const int y = idx / RW, x = idx - y * RW;
                const int gi = ry0 + y, gj = rx0 + x;
                vals[c] = 0;
                if (idx < RH * RW && gi >= 0 && gi < d.h && gj >= 0 && gj < d.w)
                    vals[c] = src[(int64_t)gi * d.pitch + gj];
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int idx = tid + (k0 + c) * NT;
                const int y = idx / RW, x = idx - y * RW;
                if (idx < RH * RW) s_img[y * RWP + x] = vals[c];
            }
        }
        return;
    }
    using V = typename std::conditional<sizeof(E) == 1, uint32_t, uint2>::type;
    constexpr int GW = RW / 4, NG = RH * GW;
    constexpr int ITER = (NG + NT - 1) / NT;
    constexpr int CH = ITER < STAGE_CHUNK ? ITER : STAGE_CHUNK;
#pragma unroll 1
    for (int k0 = 0; k0 < ITER; k0 += CH) {
        V v[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int g = tid + (k0 + c) * NT;
            const int y = g / GW, x = 4 * (g - (g / GW) * GW);
            const int gi = ry0 + y, gj = rx0 + x;
            v[c] = V{};
            if (g < NG && gi >= 0 && gi < d.h && gj >= 0 && gj < d.w) {
                const E* row = src + (int64_t)gi * d.pitch + gj;
                if (gj + 4 <= d.w) {
                    v[c] = *reinterpret_cast<const V*>(row);
                } else {
                    E q[4] = {0, 0, 0, 0};
                    for (int i = 0; i < d.w - gj; ++i) q[i] = row[i];
                    v[c] = *reinterpret_cast<const V*>(q);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int g = tid + (k0 + c) * NT;
            if (g < NG) {
                const int y = g / GW, x = 4 * (g - (g / GW) * GW);
                *reinterpret_cast<V*>(s_img + y * RWP + x) = v[c];
            }
        }
    }
}

template <typename E, int TH, int TW, int RWP, int OY, int OX, int NT>
__device__ __forceinline__ void store_native(const View& d, const void* srcv, void* dstv, int gy0,
                                             int gx0, const E* s_img, int tid)
{
    static_assert(TW % 4 == 0 && OX % 4 == 0 && RWP % 4 == 0, "groups of 4 pixels");
    E* dst = static_cast<E*>(dstv);
    const int ih = min(TH, d.h - gy0), iw = min(TW, d.w - gx0);
    if (!wide_ok(d, srcv, dstv)) {
        for (int idx = tid; idx < TH * TW; idx += NT) {
            const int y = idx / TW, x = idx - y * TW;
            if (y < ih && x < iw)
                dst[(int64_t)(gy0 + y) * d.pitch + (gx0 + x)] = s_img[(OY + y) * RWP + (OX + x)];
        }
        return;
    }
    constexpr int GW = TW / 4;
    for (int g = tid; g < TH * GW; g += NT) {
        const int y = g / GW, x = 4 * (g - (g / GW) * GW);
        if (y < ih && x < iw) {
            const E* s = s_img + (OY + y) * RWP + OX + x;
            E* q = dst + (int64_t)(gy0 + y) * d.pitch + gx0 + x;
            if (x + 4 <= iw) copy4(q, s);
            else
                for (int i = 0; i < iw - x; ++i) q[i] = s[i];
        }
    }
}

// History handed from one round to the next: for every tile processed in a
// round, a bitmap (TH rows of TW/32 words) of the interior pixels that were
// lowered during the last 4 steps of its residency, and the round it was
// written in.  Two copies alternate by round parity, so a tile of round r
// reads its neighbours' round r-1 bitmaps while they may be writing their
// round r ones.
struct Seed {
    const uint32_t* prev_bits;   // copy written in round r - 1 (unused when r == 0)
    const int32_t* prev_round;
    uint32_t* cur_bits;          // copy this round writes
    int32_t* cur_round;
    int r;                       // image-local round of the residency
    int tile0, tiles_x, tiles_y; // tile grid of the image
    int ty, tx, g;               // this tile
};

// Word `a` (global columns 32a..32a+31) of row gi of the previous round's
// change bitmaps; 0 outside the tile grid or where a tile has no bitmap for
// round r - 1 (it was skipped then, so nothing in it changed).
template <int TH, int TW>
__device__ __forceinline__ uint32_t history_word_t(const Seed* sd, int gi, int a)
{
    constexpr int WPR = TW / 32;
    if (a < 0) return 0u;
    const int tcol = a / WPR, trow = gi / TH;
    if (tcol >= sd->tiles_x || trow >= sd->tiles_y) return 0u;
    const int n = sd->tile0 + trow * sd->tiles_x + tcol;
    // both reads go out together: the bitmap of any tile of the grid may be
    // read, and is discarded unless the tile wrote it in round r - 1
    const uint32_t bits = sd->prev_bits[((int64_t)n * TH + (gi - trow * TH)) * WPR + (a - tcol * WPR)];
    return sd->prev_round[n] == sd->r - 1 ? bits : 0u;
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP moves: shifts by
// 1, 2, 4 and 8 lanes within each row of 16, then the last lane of row 0 and
// of row 2 broadcast into the next row, then lane 31 into rows 2 and 3.
// Lanes a move cannot reach add the 0 kept in `old`.
__device__ __forceinline__ int wave_inclusive_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

// The block's totals of the lanes' counts, one LDS atomic per wave and total
// (per-lane atomics on one address cost microseconds at the end of a
// residency).
__device__ __forceinline__ void block_counts(int count, int last, int exams, int* s_count,
                                             int* s_last, int* s_exam, int tid)
{
    const int c = wave_inclusive_sum(count), e = wave_inclusive_sum(exams);
    int l = last;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) l = max(l, __shfl_xor(l, o));
    if ((tid & 63) == 63) {
        if (c) {
            atomicAdd(s_count, c);
            atomicMax(s_last, l);
        }
        if (e) atomicAdd(s_exam, e);
    }
}

// Geometry of a tile residency: a TH x TW interior plus a K-pixel halo,
// staged in LDS as u16, processed by NT threads.
template <int TH, int TW, int K, int NT, bool SEED>
struct Tile {
    using Elem = uint16_t;
    static constexpr int RH = TH + 2 * K;
    static constexpr int RW = TW + 2 * K;
    static constexpr int RWP = RW;  // LDS row pitch in elements
    static constexpr int IMG_ELEMS = RH * RWP;    // LDS elements of the image tile
    static constexpr int DIRTY_ELEMS = RH * RWP;  // LDS re-examination flags
    // lanes across a candidate row: next power of two >= RW/2, at most 64
    static constexpr int LAT_H = RH / 2, LAT_W = RW / 2;  // candidate lattice of one class
    static constexpr int PPT = (LAT_H * LAT_W + NT - 1) / NT;  // lattice cells per thread
    static constexpr int WPR = TW >= 32 ? TW / 32 : 1;  // bitmap words per interior row
    static constexpr int RWW = (RW + 31) / 32;           // change-map words per region row
    // LDS words of the history arrays (one when the residency keeps no history)
    static constexpr int BITS_WORDS = SEED ? TH * WPR : 1;
    static constexpr int CW_WORDS = SEED ? RH * RWW : 1;
    static_assert(K <= TH && K <= TW, "halo must not exceed the tile side");
    static_assert(!SEED || TW % 32 == 0, "history bitmaps need a tile width multiple of 32");
    static_assert(!SEED || 2 * K <= TH, "history seeding needs the region inside the 3x3 tile block");
    static_assert(TH % 2 == 0 && TW % 2 == 0 && K % 2 == 0, "tile sides and halo must be even");


    // The change bitmap run() leaves for the tail of the visit.
    static __device__ __forceinline__ const uint32_t* changed(uint8_t*, const uint32_t* s_bits)
    {
        return s_bits;
    }

    // Tile and halo from src into s_img (no barrier).
    // Work a residency can start before the block knows whether the tile
    // runs (none for this type).
    static __device__ __forceinline__ void prefetch(const View&, int, int, const Seed*, uint8_t*,
                                                    uint32_t*, int)
    {
    }

    static __device__ __forceinline__ void stage(const View& d, int gy0, int gx0, const void* src,
                                                 const void* dst, uint16_t* s_img, int tid)
    {
        stage_region<RH, RW, RWP, 0, NT>(d, src, dst, gy0 - K, gx0 - K, s_img, tid);
    }

    // Interior of the staged tile to dst.
    static __device__ __forceinline__ void store(const View& d, int gy0, int gx0, const void* src,
                                                 void* dst, const uint16_t* s_img, int tid)
    {
        store_region<TH, TW, RWP, K, K, NT>(d, src, dst, gy0, gx0, s_img, tid);
    }

    // Runs nsteps parity steps on the tile staged by stage() (followed by a
    // barrier), starting at image step t0, and writes the interior to dst.  Returns the number of
    // interior lowerings (same value in every thread) and, in last_tau
    // (block-uniform), the last step index within the residency that lowered
    // an interior pixel (-1 if none).  Must be entered by all NT threads after
    // a barrier that ends the previous use of the shared arrays.
    //
    // A candidate is examined only when its 3x3 neighbourhood may have
    // changed since it was last examined (re-examination rule of section
    // 2.2): s_dirty starts at 1 everywhere (no history at staging), a
    // candidate clears its flag when examined, and a lowered pixel marks its
    // whole 3x3.  The decision is a function of the 3x3 only, so skipping
    // clean candidates changes nothing.  Within a step no candidate reads or
    // writes another candidate's flag: the 8 neighbours of a candidate belong
    // to other parity classes.
    //
    // With a Seed (sd != nullptr, round > 0) the flags start from history
    // instead: a candidate examined at step t0 + tau (tau < 4) was last
    // examined at step t0 + tau - 4, in the previous round, by the tile that
    // owned it (or earlier, by a tile that was then skipped because its
    // neighbourhood was quiet).  Only pixels lowered during the last 4 steps
    // of that round can have changed its 3x3 since, so the 3x3 of each such
    // pixel is marked.  The region lies inside the 3x3 tile block (K <= tile
    // side / 2), so the neighbours' bitmaps hold every pixel that matters.
    static __device__ __forceinline__ int run(const View d, int gy0, int gx0, int t0, int nsteps,
                              const void* src, void* dst, uint16_t* s_img, uint8_t* s_dirty,
                              uint32_t* s_bits, uint32_t* s_cw, const Seed* sd,
                              const DecEntry* lut, int* s_count, int* s_last, int* s_exam,
                              int tid, int& last_tau)
    {
        const int ry0 = gy0 - K, rx0 = gx0 - K;
        const bool seeded = SEED && sd != nullptr && sd->r > 0;
        if (tid == 0) {
            *s_count = 0;
            *s_last = -1;
            *s_exam = 0;
        }
        if constexpr (SEED)
            for (int i = tid; i < TH * WPR; i += NT) s_bits[i] = 0u;
        if (!seeded) {
            uint32_t* f = reinterpret_cast<uint32_t*>(s_dirty);
            for (int i = tid; i < RH * RWP / 4; i += NT) f[i] = 0x01010101u;
        }
        __syncthreads();
        if constexpr (SEED) if (seeded) {
            // Change map of the region in 32-pixel words (row y, word j covers
            // region columns 32j..32j+31), gathered from the neighbours'
            // tile-aligned bitmaps with a funnel shift, then dilated by the 3x3
            // and expanded into the byte flags.
            for (int it = tid; it < RH * RWW; it += NT) {
                const int y = it / RWW, j = it - y * RWW;
                const int gi = ry0 + y;
                uint32_t word = 0u;
                if (gi >= 0 && gi < d.h) {
                    const int c0 = rx0 + 32 * j;                  // first global column
                    const int a = (c0 >= 0) ? (c0 >> 5) : -((31 - c0) >> 5);
                    const int sh = c0 - 32 * a;                   // 0..31
                    const uint32_t lo = history_word_t<TH, TW>(sd, gi, a);
                    const uint32_t hi = history_word_t<TH, TW>(sd, gi, a + 1);
                    word = sh ? ((lo >> sh) | (hi << (32 - sh))) : lo;
                }
                s_cw[it] = word;
            }
            __syncthreads();
            for (int it = tid; it < RH * RWW; it += NT) {
                const int y = it / RWW, j = it - y * RWW;
                uint32_t m = 0u;
                for (int dy = -1; dy <= 1; ++dy) {
                    const int yy = y + dy;
                    if (yy < 0 || yy >= RH) continue;
                    const uint32_t c = s_cw[yy * RWW + j];
                    const uint32_t l = j > 0 ? s_cw[yy * RWW + j - 1] : 0u;
                    const uint32_t r = j + 1 < RWW ? s_cw[yy * RWW + j + 1] : 0u;
                    m |= c | (c << 1) | (c >> 1) | (l >> 31) | (r << 31);
                }
                uint8_t* row = s_dirty + y * RWP + 32 * j;
                const int n = min(32, RW - 32 * j);
                for (int b = 0; b < n; ++b) row[b] = (uint8_t)((m >> b) & 1u);
            }
            __syncthreads();
        }

        const Lambda lambda = lambda_of(d.lambda);
        int my_count = 0, my_last = -1;  // interior lowerings, last step with one
        int my_exams = 0;                // candidates characterised
        // Each thread owns fixed positions of the candidate lattice (one in
        // four pixels, rows and columns of the step's parity): the region's
        // origin is even (tile side and halo are even), so the candidate of
        // lattice cell (a, b) in class (si, sj) is region pixel
        // (2a + si, 2b + sj).  The exact region and the image interior only
        // mask cells out step by step.
        for (int tau = 0; tau < nsteps; ++tau) {
            const int s = (t0 + tau) & 3, si = s >> 1, sj = s & 1;
            // Exact region after tau steps, clipped to the image interior.
            const int r_lo = max(tau + 1, 1 - ry0), r_hi = min(RH - 2 - tau, d.h - 2 - ry0);
            const int c_lo = max(tau + 1, 1 - rx0), c_hi = min(RW - 2 - tau, d.w - 2 - rx0);
            bool inner = false;
            // The loop over the thread's cells stays rolled: unrolled, the
            // compiler interleaves cells and runs out of registers.
#pragma unroll 1
            for (int idx = tid; idx < LAT_H * LAT_W; idx += NT) {
                const int a = idx / LAT_W;
                const int lr = 2 * a + si, lc = 2 * (idx - a * LAT_W) + sj;
                if (lr < r_lo || lr > r_hi || lc < c_lo || lc > c_hi) continue;
                const int o = lr * RWP + lc;
                {
                    if (!s_dirty[o]) continue;
                    s_dirty[o] = 0;
                    ++my_exams;
                    uint16_t* p = s_img + o;
                    const uint32_t v = p[0];
                    const uint32_t nbv[8] = {p[1], p[-RWP + 1], p[-RWP], p[-RWP - 1],
                                             p[-1], p[RWP - 1], p[RWP], p[RWP + 1]};
                    uint32_t alpha;
                    if (decide(ring_of(v, nbv), lut, lambda, alpha)) {
                        p[0] = (uint16_t)alpha;
                        uint8_t* q = s_dirty + o;
                        q[-RWP - 1] = 1; q[-RWP] = 1; q[-RWP + 1] = 1;
                        q[-1] = 1;       q[0] = 1;    q[1] = 1;
                        q[RWP - 1] = 1;  q[RWP] = 1;  q[RWP + 1] = 1;
                        if (lr >= K && lr < K + TH && lc >= K && lc < K + TW) {
                            ++my_count;
                            inner = true;
                            if constexpr (SEED) {
                                if (tau >= nsteps - 4) {
                                    const int y = lr - K, x = lc - K;
                                    atomicOr(&s_bits[y * WPR + (x >> 5)], 1u << (x & 31));
                                }
                            }
                        }
                    }
                }
            }
            if (inner) my_last = tau;
            __syncthreads();
        }

        store(d, gy0, gx0, src, dst, s_img, tid);
        block_counts(my_count, my_last, my_exams, s_count, s_last, s_exam, tid);
        __syncthreads();
        if constexpr (SEED) {
            if (sd != nullptr) {
                for (int i = tid; i < TH * WPR; i += NT)
                    sd->cur_bits[(int64_t)sd->g * TH * WPR + i] = s_bits[i];
                if (tid == 0) sd->cur_round[sd->g] = sd->r;
            }
        }
        last_tau = *s_last;
        return *s_count;
    }
};

// Barrier for exchanges through LDS: unlike __syncthreads it does not wait
// for the wave's outstanding global stores.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Residency with register windows.  Each thread owns fixed cells of the 2x2
// lattice of the region and keeps, per cell, the 4x4 window of pixels covered
// by the 3x3 neighbourhoods of the cell's four candidates (one per parity
// class), two pixels to a register.  LDS holds the whole region as the
// exchange medium between cells and as the source of the final interior
// store.  A candidate is examined only when a pixel of its 3x3 changed since
// it was last examined (a window value re-read or received that differs, or
// the cell's own lowerings): the re-examination rule of section 2.2.
//
// What bounds it is the chain of dependent latencies of a step (read the
// neighbours, decide, look the table up, write, barrier: about 1070 cycles of
// which the barrier and the trip through LDS are 300), so:
// - steps run in phases of two, classes (0,0) and (0,1), then (1,0) and (1,1).
//   A phase changes one row of each cell, and its second class's candidates
//   touch the first class's pixels only in their own row: the cell's own and
//   the next cell's, which is the next lane's (lattice rows start at lanes
//   0, 16 or 32 of a wave), so the second step takes it with a lane shift.
//   One trip through LDS and one barrier per two steps.
// - everything beside the chain is scalar: the pending candidates of a wave's
//   cells are one 64-bit mask per class in scalar registers, updated with the
//   compare results themselves, a wave without an active candidate branches
//   past the decision, and counts are population counts of the same masks.
// With SEED the masks start from the previous round's change bitmaps (else
// every candidate starts pending), so that a quiet wave is quiet from the
// first step on.
template <int TH, int TW, int K, int NT, bool SEED>
struct RTile {
    using Elem = uint16_t;
    static constexpr int RH = TH + 2 * K;
    static constexpr int RW = TW + 2 * K;
    static constexpr int RWP = RW + 2;                // a spare column on each side
    static constexpr int IMG_ELEMS = (RH + 2) * RWP;  // a spare row above and below
    static constexpr int DIRTY_ELEMS = 4 * ((K + 7) / 8);  // "lowered" flag of each phase
    static constexpr int LAT_H = RH / 2, LAT_W = RW / 2;
    // lanes to a lattice row, and lattice cells per thread (with the lanes
    // beyond LAT_W, which hold no cell)
    static constexpr int LROW = LAT_W <= 16 ? 16 : (LAT_W <= 32 ? 32 : 64);
    static constexpr int PPT = (LAT_H * LROW + NT - 1) / NT;
    static constexpr int WPR = TW >= 32 ? TW / 32 : 1;
    static constexpr int RWW = (RW + 31) / 32;
    static constexpr int BITS_WORDS = SEED ? TH * WPR : 1;
    static constexpr int CW_WORDS = SEED ? RH * (RWW + 1) : 1;  // a zero word ends each row
    static_assert(K % 4 == 0, "a residency must start at parity class 0");
    static_assert(K <= TH && K <= TW, "halo must not exceed the tile side");
    static_assert(TH % 2 == 0 && TW % 2 == 0, "tile sides must be even");
    static_assert(RH / 2 <= 254 && RW / 2 <= 254, "step limits are bytes");
    static_assert(LAT_W <= 64 && NT % 64 == 0, "a lattice row lies in one wave");
    static_assert(TW % 4 == 0, "staged in groups of 4 pixels");

    // The lattice cell of a thread's k-th slot; false when it has none.
    static __device__ __forceinline__ bool cell(int tid, int k, int& a, int& b)
    {
        const int idx = tid + k * NT;
        a = idx / LROW;
        b = idx % LROW;
        const bool valid = a < LAT_H && b < LAT_W;
        a = valid ? a : 0;
        b = valid ? b : 0;
        return valid;
    }

    static_assert(!SEED || TW % 32 == 0, "history bitmaps need a tile width multiple of 32");
    static_assert(!SEED || 2 * K <= TH, "history seeding needs the region inside the 3x3 tile block");

    // Classes whose candidate's 3x3 contains window position (i, j); the
    // candidate of class (ci, cj) sits at (1 + ci, 1 + cj).
    static constexpr uint32_t affect(int i, int j)
    {
        uint32_t m = 0;
        for (int ci = 0; ci < 2; ++ci)
            for (int cj = 0; cj < 2; ++cj)
                if (ci <= i && i <= ci + 2 && cj <= j && j <= cj + 2) m |= 1u << (2 * ci + cj);
        return m;
    }

    // What a residency can start before the block knows whether the tile
    // runs: the step flags and, when seeded, the previous round's change map
    // of the region (read by none of the previous tile's tail).
    static __device__ __forceinline__ void prefetch(const View& d, int gy0, int gx0, const Seed* sd,
                                                    uint8_t* s_flags, uint32_t* s_cw, int tid)
    {
        if (tid < DIRTY_ELEMS / 4) reinterpret_cast<uint32_t*>(s_flags)[tid] = 0u;
        if constexpr (SEED) {
            if (sd != nullptr && sd->r > 0) {
                const int ry0 = gy0 - K, rx0 = gx0 - K;
                for (int it = tid; it < RH * (RWW + 1); it += NT) {
                    const int y = it / (RWW + 1), j = it - y * (RWW + 1);
                    const int gi = ry0 + y;
                    uint32_t word = 0u;
                    if (j < RWW && gi >= 0 && gi < d.h) {
                        const int c0 = rx0 + 32 * j;
                        const int a = (c0 >= 0) ? (c0 >> 5) : -((31 - c0) >> 5);
                        const int sh = c0 - 32 * a;
                        const uint32_t lo = history_word_t<TH, TW>(sd, gi, a);
                        const uint32_t hi = history_word_t<TH, TW>(sd, gi, a + 1);
                        word = sh ? ((lo >> sh) | (hi << (32 - sh))) : lo;
                    }
                    s_cw[it] = word;
                }
            }
        }
    }

    // The change bitmap run() leaves for the tail of the visit.
    static __device__ __forceinline__ const uint32_t* changed(uint8_t*, const uint32_t* s_bits)
    {
        return s_bits;
    }

    // Spare rows and columns zeroed (they are read into windows but never used
    // by a candidate).
    static __device__ __forceinline__ void clear_rim(uint16_t* s_img, int tid)
    {
        for (int i = tid; i < 2 * RWP + 2 * RH; i += NT) {
            int o;
            if (i < RWP) o = i;
            else if (i < 2 * RWP) o = (RH + 1) * RWP + (i - RWP);
            else if (i < 2 * RWP + RH) o = (i - 2 * RWP + 1) * RWP;
            else o = (i - 2 * RWP - RH + 1) * RWP + RWP - 1;
            s_img[o] = 0;
        }
    }

    // Tile and halo from src into s_img (no barrier), in groups of 4 pixels
    // where the buffers allow it: a quiet tile costs its staging (serving one
    // 4000x4001 image 1.50 ms, pixel by pixel 1.79).
    static __device__ __forceinline__ void stage(const View& d, int gy0, int gx0, const void* src,
                                                 const void* dst, uint16_t* s_img, int tid)
    {
        clear_rim(s_img, tid);
        stage_region<RH, RW, RWP, 1, NT>(d, src, dst, gy0 - K, gx0 - K, s_img, tid);
    }

    // The same pixel by pixel, for a kernel that stages a tile once and keeps it
    // (the groups cost k_flow 4 registers: 96 mixed images 1.972 ms, 1.960 so).
    static __device__ __forceinline__ void stage_once(const View& d, int gy0, int gx0,
                                                      const void* src, uint16_t* s_img, int tid)
    {
        clear_rim(s_img, tid);
        stage_scalar<RH, RW, RWP, 1, 1, NT>(d, src, gy0 - K, gx0 - K, s_img, tid);
    }

    static __device__ __forceinline__ void store(const View& d, int gy0, int gx0, const void* src,
                                                 void* dst, const uint16_t* s_img, int tid)
    {
        store_region<TH, TW, RWP, K + 1, K + 1, NT>(d, src, dst, gy0, gx0, s_img, tid);
    }

    struct Cells {
        uint32_t win[PPT][8];   // 4x4 windows, rows of two words
        int base[PPT];          // LDS word of window position (0, 0)
        uint32_t last[PPT];     // byte c: 1 + the last step the class-c candidate may run in
        uint64_t pend[PPT][4];  // lanes whose class-c candidate needs examining
        uint64_t inside[PPT];   // lanes whose cell is in the tile's interior
    };
    struct Counts {
        int lowered = 0, exams = 0, last = -1;  // of the wave
    };

    // Examines the active candidates of class C in step tau; the lanes whose
    // candidate of slot k was lowered.
    template <int C>
    static __device__ __forceinline__ uint64_t examine(Cells& q, int k, uint16_t* s_img,
                                                       uint32_t* s_bits, int tau, int nsteps,
                                                       int tid, const DecEntry* lut,
                                                       const Lambda& lambda, Counts& n)
    {
        constexpr int si = C >> 1, sj = C & 1, ci = 1 + si;
        const uint64_t act = q.pend[k][C] & __ballot((int)(q.last[k] >> (8 * C) & 0xFFu) > tau);
        if (act == 0) return 0;
        q.pend[k][C] &= ~act;
        uint32_t(&w)[8] = q.win[k];
        const Verdict v =
            weigh(ring_of_words<sj != 0>(w[2 * ci - 2], w[2 * ci - 1], w[2 * ci], w[2 * ci + 1],
                                         w[2 * ci + 2], w[2 * ci + 3]),
                  lut, lambda);
        const uint64_t low = act & v.lanes();
        n.exams += __popcll(act);
        if (low == 0) return 0;
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(low);
        if (mine) s_img[2 * q.base[k] + ci * RWP + 1 + sj] = (uint16_t)v.alpha;
        const uint32_t own = w[2 * ci + sj];
        const uint32_t put = sj ? ((own & 0xFFFF0000u) | v.alpha) : ((own & 0xFFFFu) | v.alpha << 16);
        w[2 * ci + sj] = mine ? put : own;
#pragma unroll
        for (int c = 0; c < 4; ++c) q.pend[k][c] |= low;
        const uint64_t in = low & q.inside[k];
        n.lowered += __popcll(in);
        n.last = in != 0 ? tau : n.last;
        if constexpr (SEED) {
            if (tau >= nsteps - 4 && __builtin_amdgcn_inverse_ballot_w64(in)) {
                int a, b;
                cell(tid, k, a, b);
                const int y = 2 * a + si - K, x = 2 * b + sj - K;
                atomicOr(&s_bits[y * WPR + (x >> 5)], 1u << (x & 31));
            }
        }
        return low;
    }

    // Steps tau and tau + 1, of classes (R, 0) and (R, 1).
    template <int R>
    static __device__ __forceinline__ void phase(Cells& q, uint16_t* s_img, uint8_t* s_flags,
                                                 uint32_t* s_bits, int tau, int nsteps, int tid,
                                                 const DecEntry* lut, const Lambda& lambda,
                                                 Counts& n)
    {
        const uint32_t* words = reinterpret_cast<const uint32_t*>(s_img);
        if (tau > 0) {
            // The phase before changed the pixel rows of the other parity: in
            // the window the cell's own row of it (columns 0 and 3 belong to
            // other cells) and one row of the cells above or below.  No row
            // read here is written in this phase.
            constexpr int own = R ? 1 : 2, far = R ? 3 : 0;
            constexpr int fi = R ? 1 : 0;  // the classes whose 3x3 holds that row
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                uint32_t now[4], x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    now[e] = words[q.base[k] + (e < 2 ? own : far) * (RWP / 2) + (e & 1)];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t& w = q.win[k][2 * (e < 2 ? own : far) + (e & 1)];
                    x[e] = now[e] ^ w;
                    w = now[e];
                }
                const uint64_t left = __ballot(x[0] != 0u), right = __ballot(x[1] != 0u);
                // columns 0..2 of the far row touch (fi, 0), columns 1..3 (fi, 1)
                const uint64_t f0 = __ballot((x[2] | (x[3] & 0xFFFFu)) != 0u);
                const uint64_t f1 = __ballot((x[3] | x[2] >> 16) != 0u);
                q.pend[k][0] |= left;
                q.pend[k][2] |= left;
                q.pend[k][1] |= right;
                q.pend[k][3] |= right;
                q.pend[k][2 * fi] |= f0;
                q.pend[k][2 * fi + 1] |= f1;
            }
        }
        uint64_t any = 0;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const uint64_t low =
                examine<2 * R>(q, k, s_img, s_bits, tau, nsteps, tid, lut, lambda, n);
            if (low == 0) continue;
            any |= low;
            // the next cell's (R, 0) pixel is this window's column 3
            const uint32_t mine = q.win[k][2 * (1 + R)];
            const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(
                (int)mine, (int)mine, 0x130, 0xf, 0xf, false);  // wave_shl:1
            const uint32_t was = q.win[k][2 * (1 + R) + 1];
            const uint32_t now = (next & 0xFFFF0000u) | (was & 0xFFFFu);
            const uint64_t right = __ballot(now != was);
            q.win[k][2 * (1 + R) + 1] = now;
            q.pend[k][1] |= right;
            q.pend[k][3] |= right;
        }
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            any |= examine<2 * R + 1>(q, k, s_img, s_bits, tau + 1, nsteps, tid, lut, lambda, n);
        if (any != 0 && (tid & 63) == 0) s_flags[tau >> 1] = 1;
        lds_barrier();
    }

    // Windows of the staged region, every candidate pending (no barrier).
    static __device__ __forceinline__ void open(Cells& q, const View& d, int gy0, int gx0,
                                                const uint16_t* s_img, int tid)
    {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            int a, b;
            const bool valid = cell(tid, k, a, b);
            q.base[k] = a * RWP + b;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t* row = reinterpret_cast<const uint32_t*>(s_img) + q.base[k] + i * (RWP / 2);
                q.win[k][2 * i] = row[0];
                q.win[k][2 * i + 1] = row[1];
            }
            // A class-(si, sj) candidate at region pixel (lr, lc) may run in
            // step tau while it lies tau + 1 pixels inside the region, and
            // only in the image's interior.
            uint32_t last = 0u;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int lr = 2 * a + (c >> 1), lc = 2 * b + (c & 1);
                const int in = min(min(lr, RH - 1 - lr), min(lc, RW - 1 - lc));
                const int gi = gy0 - K + lr, gj = gx0 - K + lc;
                const bool ok = valid && gi >= 1 && gi <= d.h - 2 && gj >= 1 && gj <= d.w - 2;
                last |= (ok ? (uint32_t)in : 0u) << (8 * c);
            }
            q.last[k] = last;
            const bool inside = valid && 2 * a >= K && 2 * a < K + TH && 2 * b >= K && 2 * b < K + TW;
            q.inside[k] = __ballot(inside);
#pragma unroll
            for (int c = 0; c < 4; ++c) q.pend[k][c] = ~0ull;
        }
    }

    // Pending candidates from the previous round's change map instead.
    static __device__ __forceinline__ void seed(Cells& q, const uint32_t* s_cw, int tid)
    {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            int a, b;
            cell(tid, k, a, b);
            // the change map over the cell's window, rows 2a - 1 .. 2a + 2
            // (clamped: candidates of the region's rim never run), columns
            // 2b - 1 .. 2b + 2 in bits 0..3
            uint32_t m[4];
            const int col = 2 * b, wj = col >> 5, sh = col & 31;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int y = min(max(2 * a - 1 + i, 0), RH - 1);
                const uint32_t* row = s_cw + y * (RWW + 1) + wj;
                const uint64_t two = ((uint64_t)row[1] << 32 | row[0]) << 1;
                // column 2b - 1 is the last bit of the word before when 2b
                // starts a word
                const uint32_t carry = sh == 0 && wj > 0 ? row[-1] >> 31 : 0u;
                m[i] = (uint32_t)(two >> sh) | carry;
            }
            const uint32_t up = m[0] | m[1] | m[2], down = m[1] | m[2] | m[3];
            q.pend[k][0] = __ballot((up & 0x7u) != 0u);
            q.pend[k][1] = __ballot((up & 0xEu) != 0u);
            q.pend[k][2] = __ballot((down & 0x7u) != 0u);
            q.pend[k][3] = __ballot((down & 0xEu) != 0u);
        }
    }

    // Windows from the region's current values: a candidate whose 3x3 holds a
    // value that differs becomes pending (no barrier).
    static __device__ __forceinline__ void refresh(Cells& q, const uint16_t* s_img)
    {
        const uint32_t* words = reinterpret_cast<const uint32_t*>(s_img);
#pragma unroll
        for (int k = 0; k < PPT; ++k)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int i = e >> 1, w = e & 1;
                const uint32_t now = words[q.base[k] + i * (RWP / 2) + w];
                const uint64_t changed = __ballot(now != q.win[k][e]);
                q.win[k][e] = now;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if ((affect(i, 2 * w) | affect(i, 2 * w + 1)) >> c & 1u) q.pend[k][c] |= changed;
            }
    }

    // nsteps steps (a multiple of 4) from class 0 on, ending in a barrier
    // (s_flags cleared and s_img complete before).
    static __device__ __forceinline__ void steps(Cells& q, uint16_t* s_img, uint8_t* s_flags,
                                                 uint32_t* s_bits, int nsteps, int tid,
                                                 const DecEntry* lut, const Lambda& lambda,
                                                 Counts& n)
    {
        for (int tau = 0; tau < nsteps; tau += 4) {
            // four quiet steps: nothing in the region can change any more
            // (candidates left pending lie outside the exact region for good)
            if (tau > 0 && __builtin_amdgcn_readfirstlane(
                               (int)reinterpret_cast<const uint16_t*>(s_flags)[tau / 4 - 1]) == 0)
                break;
            phase<0>(q, s_img, s_flags, s_bits, tau, nsteps, tid, lut, lambda, n);
            phase<1>(q, s_img, s_flags, s_bits, tau + 2, nsteps, tid, lut, lambda, n);
        }
    }

    // Same contract as Tile::run.
    static __device__ __forceinline__ int run(const View d, int gy0, int gx0, int t0, int nsteps,
                              const void* src, void* dst, uint16_t* s_img, uint8_t* s_flags,
                              uint32_t* s_bits, uint32_t* s_cw, const Seed* sd,
                              const DecEntry* lut, int* s_count, int* s_last, int* s_exam, int tid,
                              int& last_tau)
    {
        (void)t0;  // a multiple of 4: step tau has class tau mod 4
        const bool seeded = SEED && sd != nullptr && sd->r > 0;
        if (tid == 0) {
            *s_count = 0;
            *s_last = -1;
            *s_exam = 0;
        }
        if constexpr (SEED)
            for (int i = tid; i < TH * WPR; i += NT) s_bits[i] = 0u;
        // The barrier after the windows are read also orders the resets above
        // before the steps' updates.
        Cells q;
        open(q, d, gy0, gx0, s_img, tid);
        if constexpr (SEED)
            if (seeded) seed(q, s_cw, tid);
        __syncthreads();

        Counts n;
        steps(q, s_img, s_flags, s_bits, nsteps, tid, lut, lambda_of(d.lambda), n);

        store(d, gy0, gx0, src, dst, s_img, tid);
        if ((tid & 63) == 0) {
            if (n.lowered) {
                atomicAdd(s_count, n.lowered);
                atomicMax(s_last, n.last);
            }
            if (n.exams) atomicAdd(s_exam, n.exams);
        }
        __syncthreads();
        if constexpr (SEED) {
            if (sd != nullptr) {
                for (int i = tid; i < TH * WPR; i += NT)
                    sd->cur_bits[(int64_t)sd->g * TH * WPR + i] = s_bits[i];
                if (tid == 0) sd->cur_round[sd->g] = sd->r;
            }
        }
        last_tau = *s_last;
        return *s_count;
    }
};

// Residency with bit flags and dense work lists.  "Lowered" bitmaps hold, one
// bit per lattice cell and parity class (4 x LAT_H rows of LWW words), the
// cells lowered by that class's latest step; the candidates to examine from
// the residency's start (all of them, or with SEED those next to the previous
// round's change bitmaps) stay in the registers of the lanes that own their
// words.  A step of class c needs the candidates whose 3x3 changed since
// their examination 4 steps earlier (section 2.2 re-examination rule): the
// cell itself if it was lowered then, and any pixel of its 3x3 lowered by the
// 3 steps since, one class each; the owner of each bitmap word gathers those
// from the lowered bitmaps with word shifts (pull), so a lowering costs one
// LDS atomic.  Every wave takes the candidates of its run of words and writes
// them into a run of the step's list that it reserves with one LDS atomic, at
// offsets from a wave prefix sum; after one barrier the block examines the
// list densely, so clean candidates cost nothing beyond their share of one
// word.
// The seeded start: a candidate whose 3x3 saw none of the pixels lowered
// during the last 4 steps of round r - 1 (dilated by the 3x3) was examined 4
// steps earlier at the same values.
//
// What bounds it: in the dense first round the vector units (85 % of their
// issue slots in 8 bits; per 64 examinations 58 instructions in 16 bits and 51 in 8, per
// wave and step about 170 for gather and list), later the chain of a tile's
// few busy steps.  (63 and 67 with the 16-bit decision for both and lanes'
// verdicts joined in registers: 512 images, 162 Mpx in all, in 8 bits 6.72 ms,
// now 6.35; 8192x8192 in 16 bits 1.554, now 1.518.)
template <int TH, int TW, int K, int NT, bool SEED, typename E>
struct BTile {
    using Elem = E;  // LDS pixel type: the image's own
    static constexpr int RH = TH + 2 * K;
    static constexpr int RW = TW + 2 * K;
    static constexpr int RWP = RW;
    // the widened reads of the last candidate reach a pixel past the region
    static constexpr int IMG_ELEMS = RH * RWP + 4;
    static constexpr int LAT_H = RH / 2, LAT_W = RW / 2;
    static constexpr int NCELL = LAT_H * LAT_W;
    static constexpr int LWW = (LAT_W + 31) / 32;     // bitmap words per lattice row
    static constexpr int CLASS_WORDS = LAT_H * LWW;   // bitmap words per class
    static constexpr int NWAVE = NT / 64;
    // Bitmap words of a class are dealt to the waves in runs of WAVE_WORDS
    // (whole lattice rows), so each wave's run of the list is in raster order
    // and neighbouring lanes examine neighbouring cells.  Where the run leaves
    // half the lanes idle, two lanes share a word, half of its bits each: a
    // lane's part of the list is written bit by bit.
    static constexpr int WAVE_ROWS = (LAT_H + NWAVE - 1) / NWAVE;
    static constexpr int WAVE_WORDS = WAVE_ROWS * LWW;
    static constexpr int SPLIT = WAVE_WORDS <= 32 ? 2 : 1;  // lanes to a word
    static constexpr int LIST_ELEMS = (NCELL + 1) & ~1;
    static constexpr int WPR = TW >= 32 ? TW / 32 : 1;
    static constexpr int RWW = (RW + 31) / 32;
    // LDS words behind the flag pointer: a pad (reads one row and word before
    // the bitmaps), 4 lowered bitmaps, a ring of 8 list lengths and 8
    // "lowered" flags (by step), 4 "has seeds" flags (by class), the step's
    // list.  Outside the steps the list's space holds the change bitmap
    // handed to the next round and, behind it, the previous round's change
    // map of the next tile (whose staging may overlap this tile's tail).
    static constexpr int PAD_WORDS = LWW + 1;
    static constexpr int LIST_AT = PAD_WORDS + 4 * CLASS_WORDS + 8 + 4;
    static constexpr int CHANGED_WORDS = SEED ? TH * WPR : 0;
    static constexpr int MAP_WORDS = SEED ? RH * RWW : 0;
    static constexpr int LIST_WORDS = LIST_ELEMS / 2 > CHANGED_WORDS + MAP_WORDS
                                          ? LIST_ELEMS / 2 : CHANGED_WORDS + MAP_WORDS;
    static constexpr int DIRTY_ELEMS = 4 * (LIST_AT + LIST_WORDS);
    static constexpr int BITS_WORDS = 1, CW_WORDS = 1;
    static_assert(K % 4 == 0, "a residency must start at parity class 0");
    static_assert(K <= TH && K <= TW, "halo must not exceed the tile side");
    static_assert(TH % 4 == 0 && TW % 4 == 0, "tile sides must be multiples of 4");
    static_assert(NT % 64 == 0 && CLASS_WORDS <= NT, "one bitmap word per thread");
    static_assert(WAVE_WORDS <= 64, "at most one bitmap word per lane");
    static_assert(LWW + 1 <= 8, "reads one row and word past the lowered bitmaps stay in the ring");
    static_assert(LAT_H <= 256 && LAT_W <= 256, "list entries hold a row and a column byte");
    static_assert(!SEED || TW % 32 == 0, "history bitmaps need a tile width multiple of 32");
    static_assert(!SEED || 2 * K <= TH, "history seeding needs the region inside the 3x3 tile block");


    // The flag area's parts.
    static __device__ __forceinline__ uint32_t* lowered_maps(uint8_t* s_flags)
    {
        return reinterpret_cast<uint32_t*>(s_flags) + PAD_WORDS;
    }
    static __device__ __forceinline__ uint32_t* list_words(uint8_t* s_flags)
    {
        return reinterpret_cast<uint32_t*>(s_flags) + LIST_AT;
    }
    // The change bitmap run() leaves for the tail of the visit.
    static __device__ __forceinline__ const uint32_t* changed(uint8_t* s_flags, const uint32_t*)
    {
        return list_words(s_flags);
    }

    // Everything a residency can start before the block knows whether the
    // tile runs, so that it overlaps the staging loads instead of following
    // them: the ring slots and flags, the cleared lowered bitmaps and, when
    // seeded, the previous round's change map of the region in 32-pixel words.
    // None of it is read by the previous tile's tail.
    static __device__ __forceinline__ void prefetch(const View& d, int gy0, int gx0, const Seed* sd,
                                                    uint8_t* s_flags, uint32_t*, int tid)
    {
        uint32_t* s_dl = lowered_maps(s_flags);
        int* s_total = reinterpret_cast<int*>(s_dl + 4 * CLASS_WORDS);
        uint8_t* s_low = reinterpret_cast<uint8_t*>(s_total + 8);
        uint8_t* s_seeds = s_low + 8;
        const bool seeded = SEED && sd != nullptr && sd->r > 0;
        for (int i = tid; i < 4 * CLASS_WORDS; i += NT) s_dl[i] = 0u;
        if (tid < 8) {
            s_total[tid] = 0;
            s_low[tid] = 0;
            if (tid < 4) s_seeds[tid] = seeded ? 0 : 1;
        }
        if constexpr (SEED) {
            if (seeded) {
                uint32_t* map = list_words(s_flags) + CHANGED_WORDS;
                const int ry0 = gy0 - K, rx0 = gx0 - K;
                for (int it = tid; it < RH * RWW; it += NT) {
                    const int y = it / RWW, j = it - y * RWW;
                    const int gi = ry0 + y;
                    uint32_t word = 0u;
                    if (gi >= 0 && gi < d.h) {
                        const int c0 = rx0 + 32 * j;
                        const int a = (c0 >= 0) ? (c0 >> 5) : -((31 - c0) >> 5);
                        const int sh = c0 - 32 * a;
                        const uint32_t lo = history_word_t<TH, TW>(sd, gi, a);
                        const uint32_t hi = history_word_t<TH, TW>(sd, gi, a + 1);
                        word = sh ? ((lo >> sh) | (hi << (32 - sh))) : lo;
                    }
                    map[it] = word;
                }
            }
        }
    }

    static __device__ __forceinline__ void stage(const View& d, int gy0, int gx0, const void* src,
                                                 const void* dst, E* s_img, int tid)
    {
        stage_native<E, RH, RW, RWP, NT>(d, src, dst, gy0 - K, gx0 - K, s_img, tid);
    }

    static __device__ __forceinline__ void store(const View& d, int gy0, int gx0, const void* src,
                                                 void* dst, const E* s_img, int tid)
    {
        store_native<E, TH, TW, RWP, K, K, NT>(d, src, dst, gy0, gx0, s_img, tid);
    }

    // Bits of lattice word j that exist (cells b < LAT_W).
    static __device__ __forceinline__ uint32_t valid_bits(int j)
    {
        constexpr int tail = LAT_W - 32 * (LWW - 1);
        return (j < LWW - 1 || tail == 32) ? ~0u : ((1u << tail) - 1u);
    }

    // Even bits of x packed into the low 16 bits.
    static __device__ __forceinline__ uint32_t even_bits(uint32_t x)
    {
        x &= 0x55555555u;
        x = (x | (x >> 1)) & 0x33333333u;
        x = (x | (x >> 2)) & 0x0F0F0F0Fu;
        x = (x | (x >> 4)) & 0x00FF00FFu;
        x = (x | (x >> 8)) & 0x0000FFFFu;
        return x;
    }

    // The low 16 bits of x at the even bits of the result.
    static __device__ __forceinline__ uint32_t spread_bits(uint32_t x)
    {
        x &= 0xFFFFu;
        x = (x | (x << 8)) & 0x00FF00FFu;
        x = (x | (x << 4)) & 0x0F0F0F0Fu;
        x = (x | (x << 2)) & 0x33333333u;
        return (x | (x << 1)) & 0x55555555u;
    }

    // Same contract as Tile::run.
    static __device__ __forceinline__ int run(const View d, int gy0, int gx0, int t0, int nsteps,
                                              const void* src, void* dst, E* s_img,
                                              uint8_t* s_flags, uint32_t*, uint32_t*,
                                              const Seed* sd, const DecEntry* lut, int* s_count,
                                              int* s_last, int* s_exam, int tid, int& last_tau)
    {
        (void)t0;  // a multiple of 4: step tau has class tau mod 4
        uint32_t* s_dl = lowered_maps(s_flags);                          // [4][LAT_H][LWW]
        int* s_total = reinterpret_cast<int*>(s_dl + 4 * CLASS_WORDS);   // [8]: step tau & 7
        uint8_t* s_low = reinterpret_cast<uint8_t*>(s_total + 8);        // [8]: step tau & 7
        uint8_t* s_seeds = s_low + 8;                                    // [4]: class
        uint16_t* s_list = reinterpret_cast<uint16_t*>(list_words(s_flags));
        const int ry0 = gy0 - K, rx0 = gx0 - K;
        const bool seeded = SEED && sd != nullptr && sd->r > 0;
        if (tid == 0) {
            *s_count = 0;
            *s_last = -1;
            *s_exam = 0;
        }
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        // The bitmap word this lane owns, and its bits of it; lanes without
        // one read a valid word (the last) and take nothing.  Every read of a
        // step is unconditional, so a step's reads go out together: a word of
        // a neighbouring row or column outside the lattice reads some other
        // word of the flag area (they all lie inside it) and is masked to zero.
        const int part = lane % SPLIT;
        const bool has_word =
            lane / SPLIT < WAVE_WORDS && wave * WAVE_WORDS + lane / SPLIT < CLASS_WORDS;
        const int myw = has_word ? wave * WAVE_WORDS + lane / SPLIT : CLASS_WORDS - 1;
        const int wa = myw / LWW, wj = myw - (myw / LWW) * LWW;
        const bool up_ok = wa > 0, dn_ok = wa + 1 < LAT_H, lt_ok = wj > 0, rt_ok = wj + 1 < LWW;
        const uint32_t mine = !has_word ? 0u
                              : SPLIT == 1 ? valid_bits(wj)
                                           : valid_bits(wj) & (part ? 0xFFFF0000u : 0x0000FFFFu);
        uint32_t seeds[4] = {mine, mine, mine, mine};  // by class, pending since the start
        if constexpr (SEED) if (seeded) {
            // Bits 16h .. 16h + 15 of word j of class (si, sj) cover region
            // row 2a + si, columns 64j + 32h + sj + 2t: the 3x3-dilated change
            // map there (its word 2j + h), odd or even columns packed.  Every
            // read is unconditional (clamped into the map, the value masked),
            // so all of them go out together.
            const uint32_t* map = list_words(s_flags) + CHANGED_WORDS;
#pragma unroll
            for (int c = 0; c < 4; ++c) seeds[c] = 0u;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (SPLIT == 2 && h > 0) break;
                const int half = SPLIT == 2 ? part : h;
                const int w = 2 * wj + half;
                const int wc = w < RWW ? w : RWW - 1;
                const int wl = wc > 0 ? wc - 1 : 0, wr = wc + 1 < RWW ? wc + 1 : wc;
                uint32_t row[4];  // dilated along the row: region rows 2a - 1 .. 2a + 2
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int yy = 2 * wa - 1 + e;
                    const int yc = yy < 0 ? 0 : (yy >= RH ? RH - 1 : yy);
                    const uint32_t cc = map[yc * RWW + wc];
                    const uint32_t l = map[yc * RWW + wl], r = map[yc * RWW + wr];
                    const uint32_t m = cc | (cc << 1) | (cc >> 1) | (wc > 0 ? l >> 31 : 0u) |
                                       (wc + 1 < RWW ? r << 31 : 0u);
                    row[e] = (yy >= 0 && yy < RH && w < RWW) ? m : 0u;
                }
                const uint32_t m0 = row[0] | row[1] | row[2], m1 = row[1] | row[2] | row[3];
                seeds[0] |= even_bits(m0) << (16 * half);
                seeds[1] |= even_bits(m0 >> 1) << (16 * half);
                seeds[2] |= even_bits(m1) << (16 * half);
                seeds[3] |= even_bits(m1 >> 1) << (16 * half);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                seeds[c] &= mine;
                if (seeds[c]) s_seeds[c] = 1;
            }
        }
        __syncthreads();

        const Lambda lambda = lambda_of(sizeof(E) == 1 ? min(d.lambda, 255u) : d.lambda);
        const uint32_t* own_dl = s_dl + myw;  // word (wa, wj) of class 0's lowered bitmap
        int my_count = 0, my_last = -1;  // the wave's interior lowerings, last step with one
        int my_exams = 0;                // candidates characterised (the block's)
        bool done = false;               // block-uniform: no later step can lower anything

        // One step of class C = tau mod 4.  A step's candidates come from the
        // residency's seeds (first 4 steps) and from pixels lowered during the
        // 4 steps before it.  When neither exists the step cannot lower
        // anything; once 4 steps in a row are quiet and the seeds are used up,
        // no later step of the residency can either.  The flags were written
        // before the last barrier, so every thread takes the same branch.  A
        // skipped step still clears the two ring slots it owns (its "lowered"
        // flag, and the list length of step tau + 4, whose last readers were
        // at step tau - 4).
        auto step = [&](auto cls, int tau) __attribute__((always_inline)) {
            constexpr int c = decltype(cls)::value, si = c >> 1, sj = c & 1;
            const uint32_t* flags = reinterpret_cast<const uint32_t*>(s_low);
            const uint32_t lw0 = flags[0], lw1 = flags[1], lws = flags[2];
            // Candidates of this word: still pending from the residency's
            // start, lowered themselves 4 steps ago, or next to a pixel
            // lowered during the last 3 steps (the lowered bitmap of each
            // other class, spread over the cells whose 3x3 holds it: rows a
            // or a+-1 and columns b or b+-1 by parity).  Read before the quiet
            // test; in a quiet step every one of these words is zero.
            uint32_t want = seeds[c] | own_dl[c * CLASS_WORDS];
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                const int o = (c + k) & 3, oi = o >> 1, oj = o & 1;
                const uint32_t* bm = own_dl + o * CLASS_WORDS;  // word (wa, wj) of class o
                // rows of o next to row wa of c: wa itself when oi == si, else
                // wa - 1 and wa (oi > si) or wa and wa + 1 (oi < si)
                const int dr = oi > si ? -LWW : LWW;
                const bool r_ok = oi > si ? up_ok : dn_ok;
                uint32_t w0 = bm[0], prev = 0u, next = 0u;
                if (oj > sj) prev = bm[-1];
                if (oj < sj) next = bm[1];
                if (oi != si) {
                    const uint32_t x0 = bm[dr];
                    const uint32_t xp = oj > sj ? bm[dr - 1] : 0u;
                    const uint32_t xn = oj < sj ? bm[dr + 1] : 0u;
                    w0 |= r_ok ? x0 : 0u;
                    prev |= r_ok ? xp : 0u;
                    next |= r_ok ? xn : 0u;
                }
                if (oj == sj) {
                    want |= w0;
                } else if (oj > sj) {  // cells b - 1 and b
                    want |= w0 | (w0 << 1) | ((lt_ok ? prev : 0u) >> 31);
                } else {               // cells b and b + 1
                    want |= w0 | (w0 >> 1) | ((rt_ok ? next : 0u) << 31);
                }
            }
            {
                // "lowered" flags of steps tau - 4 .. tau - 1: the ring's half
                // that holds the group of 4 steps before, and the steps of
                // this group in the other
                const uint32_t half0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lw0);
                const uint32_t half1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lw1);
                const bool seeds_c = ((uint32_t)__builtin_amdgcn_readfirstlane((int)lws) >> (8 * c) & 0xFFu) != 0;
                const uint32_t now = tau & 4 ? half1 : half0, before = tau & 4 ? half0 : half1;
                const uint32_t recent = (now & ((1u << (8 * c)) - 1u)) | (before >> (8 * c));
                if (recent == 0u && !(tau < 4 && seeds_c)) {
                    if (tau >= 4) {
                        done = true;
                        return;
                    }
                    if (tid == 0) {
                        s_low[tau & 7] = 0;
                        s_total[(tau + 4) & 7] = 0;
                    }
                    return;
                }
            }
            if (tid == 0) s_low[tau & 7] = 0;
            seeds[c] = 0u;
            if (has_word) s_dl[c * CLASS_WORDS + myw] = 0u;
            // Exact region after tau steps, clipped to the image interior,
            // as lattice rows a (region row 2a + si) and columns b (2b + sj).
            const int r_lo = max(tau + 1, 1 - ry0), r_hi = min(RH - 2 - tau, d.h - 2 - ry0);
            const int c_lo = max(tau + 1, 1 - rx0), c_hi = min(RW - 2 - tau, d.w - 2 - rx0);
            const int a_lo = (r_lo - si + 1) >> 1, a_hi = (r_hi - si) >> 1;
            const int b_lo = (c_lo - sj + 1) >> 1, b_hi = (c_hi - sj) >> 1;
            uint32_t take = 0u;
            {
                const int lo = max(b_lo - 32 * wj, 0), hi = min(b_hi - 32 * wj, 31);
                if (wa >= a_lo && wa <= a_hi && lo <= hi) {
                    const uint32_t mask = (hi == 31 ? ~0u : ((2u << hi) - 1u)) & ~((1u << lo) - 1u);
                    take = want & mask & mine;
                }
            }
            // Each wave reserves a run of the step's list with one LDS atomic
            // (the counter of the other parity was read a step ago and is
            // cleared for the next step while this one is examined).
            const int cnt = __popc(take);
            const int incl = wave_inclusive_sum(cnt);
            const int wave_total = __builtin_amdgcn_readlane(incl, 63);
            int base = 0;
            if (lane == 63 && wave_total) base = atomicAdd(&s_total[tau & 7], wave_total);
            base = __builtin_amdgcn_readlane(base, 63);
            if (take) {
                int off = base + incl - cnt;
                uint32_t t = take;
                while (t) {
                    // entry: lattice row in the high byte, column in the low
                    s_list[off++] = (uint16_t)((wa << 8) | (32 * wj + __ffs(t) - 1));
                    t &= t - 1u;
                }
            }
            __syncthreads();
            // Every wave takes 64 entries at a time; past the end of the list
            // its lanes repeat the last entry and are masked.  The loop, the
            // verdicts and the counts are the wave's (scalar), so a lane's
            // work is the decision and its own writes.
            const int total = __builtin_amdgcn_readfirstlane(s_total[tau & 7]);
            if (tid == 0) s_total[(tau + 4) & 7] = 0;
            bool lowered = false;
            const uint8_t* list = reinterpret_cast<const uint8_t*>(s_list);
            auto entry = [&](int byte) { return (int)*reinterpret_cast<const uint16_t*>(list + byte); };
            int at = 2 * tid;  // this lane's entry, in bytes
            int next_cell = entry(min(at, max(2 * total - 2, 0)));
            for (int i0 = 64 * wave; i0 < total; i0 += NT, at += 2 * NT) {
                const int cell = next_cell;
                next_cell = entry(min(at + 2 * NT, 2 * total - 2));
                const int a = cell >> 8, b = cell & 0xFF;
                const int o = (2 * a + si) * RWP + 2 * b + sj;
                // the words around W, centre, E of the three rows, all read
                // before the first is used (left to itself the compiler,
                // short of registers, waits for each row in turn)
                uint32_t w[6];
                Ring q;
                if constexpr (sizeof(E) == 1) {
                    const int x0 = o - RWP - 1;  // (addressed from the row above: no negative offset)
                    const uint32_t* row = reinterpret_cast<const uint32_t*>(s_img) + (x0 >> 2);
#pragma unroll
                    for (int y = 0; y < 6; ++y) w[y] = row[(y / 2) * (RWP / 4) + (y & 1)];
                    asm("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]));
                    // (unaligned LDS reads cost more than the funnel shift)
                    q = ring_of_bytes(__builtin_amdgcn_alignbyte(w[1], w[0], x0 & 3),
                                      __builtin_amdgcn_alignbyte(w[3], w[2], x0 & 3),
                                      __builtin_amdgcn_alignbyte(w[5], w[4], x0 & 3));
                } else {
                    // an even column is the third of its four pixels
                    const uint32_t* row =
                        reinterpret_cast<const uint32_t*>(s_img + o - RWP - (sj ? 1 : 2));
#pragma unroll
                    for (int y = 0; y < 6; ++y) w[y] = row[(y / 2) * (RWP / 2) + (y & 1)];
                    asm("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]));
                    q = ring_of_words<sj == 0>(w[0], w[1], w[2], w[3], w[4], w[5]);
                }
                const Verdict v = sizeof(E) == 1 ? weigh_small(q, lut, lambda) : weigh(q, lut, lambda);
                const uint64_t low = __ballot(at < 2 * total) & v.lanes();
                if (low == 0) continue;
                lowered = true;
                // in the tile's interior, as one compare per axis
                const uint64_t in = low & __ballot((uint32_t)(a - K / 2) < (uint32_t)(TH / 2)) &
                                    __ballot((uint32_t)(b - K / 2) < (uint32_t)(TW / 2));
                if (__builtin_amdgcn_inverse_ballot_w64(low)) {
                    s_img[o] = (E)v.alpha;
                    atomicOr(&s_dl[c * CLASS_WORDS + a * LWW + (b >> 5)], 1u << (b & 31));
                }
                my_count += __popcll(in);
                my_last = in != 0 ? tau : my_last;
            }
            my_exams += total;
            if (lowered && lane == 0) s_low[tau & 7] = 1;
            __syncthreads();
        };
        using C0 = std::integral_constant<int, 0>;
        using C1 = std::integral_constant<int, 1>;
        using C2 = std::integral_constant<int, 2>;
        using C3 = std::integral_constant<int, 3>;
        for (int tau = 0; tau < nsteps && !done; tau += 4) {
            step(C0{}, tau);
            if (tau + 1 < nsteps && !done) step(C1{}, tau + 1);
            if (tau + 2 < nsteps && !done) step(C2{}, tau + 2);
            if (tau + 3 < nsteps && !done) step(C3{}, tau + 3);
        }

        store(d, gy0, gx0, src, dst, s_img, tid);
        if (lane == 0) {
            if (my_count) {
                atomicAdd(s_count, my_count);
                atomicMax(s_last, my_last);
            }
            if (wave == 0) *s_exam = my_exams;
        }
        if constexpr (SEED) {
            // The interior pixels lowered during the last 4 steps, in pixel
            // order: exactly what the lowered bitmaps hold now (one step of
            // each class; a skipped step's class lowered nothing in its last
            // one).  Word w of interior row y: 16 cells from column K/2 + 16w.
            uint32_t* out = list_words(s_flags);
            for (int i = tid; i < TH * WPR; i += NT) {
                const int y = i / WPR, w = i - y * WPR;
                const int a = (K + y) >> 1, b0 = K / 2 + 16 * w, j = b0 >> 5, sh = b0 & 31;
                const uint32_t* even = s_dl + (2 * (y & 1)) * CLASS_WORDS + a * LWW + j;
                const uint32_t* odd = even + CLASS_WORDS;
                // 16 bits from bit sh of word j (and its successor)
                const uint32_t e = (uint32_t)((((uint64_t)even[1] << 32) | even[0]) >> sh);
                const uint32_t o = (uint32_t)((((uint64_t)odd[1] << 32) | odd[0]) >> sh);
                const uint32_t bits = spread_bits(e) | spread_bits(o) << 1;
                out[i] = bits;
                if (sd != nullptr) sd->cur_bits[(int64_t)sd->g * TH * WPR + i] = bits;
            }
            if (sd != nullptr && tid == 0) sd->cur_round[sd->g] = sd->r;
        }
        __syncthreads();
        last_tau = *s_last;
        return *s_count;
    }
};

// Residency type of a variant; E is the LDS pixel type of the bit-flag
// variants (the other variants keep u16).
template <int TH, int TW, int K, int NT, int VAR, typename E = uint16_t>
using TileOf = typename std::conditional<
    VAR == kVarRegs || VAR == kVarRegsSeeded, RTile<TH, TW, K, NT, VAR == kVarRegsSeeded>,
    typename std::conditional<VAR == kVarBits || VAR == kVarBitsSeeded,
                              BTile<TH, TW, K, NT, VAR == kVarBitsSeeded, E>,
                              Tile<TH, TW, K, NT, VAR == kVarSeeded>>::type>::type;

// Waves per SIMD that the LDS of one residency of T allows (blocks per CU
// times waves per block over the 4 SIMDs).  The large bit-flag tiles of the
// batched path ask the compiler to fit their registers to it, so that
// register growth never costs them a resident block (their register needs
// sit just under that budget); the other shapes need more registers than
// their LDS occupancy would leave them, and ask for nothing (1).
template <typename T, int NT, int TH, int VAR>
constexpr int lds_waves_per_eu()
{
    if constexpr (!(TH >= 128 && (VAR == kVarBits || VAR == kVarBitsSeeded))) return 1;
    constexpr int lds = (int)sizeof(typename T::Elem) * T::IMG_ELEMS + T::DIRTY_ELEMS +
                        4 * T::BITS_WORDS + 4 * T::CW_WORDS + (int)sizeof(DecEntry) * 256 + 64;
    constexpr int by_lds = (160 * 1024) / lds;
    constexpr int by_threads = 2048 / NT;
    constexpr int blocks = by_lds < by_threads ? by_lds : by_threads;
    constexpr int w = (blocks < 1 ? 1 : blocks) * (NT / 64) / 4;
    return w < 1 ? 1 : (w > 8 ? 8 : w);
}

// ----------------------------------------------------------------- k_round

// One tile of one round (launch-per-round and cooperative engines).
// Returns 1 when the tile was processed (active), 0 when skipped.  All NT
// threads must call it together.
// Queues tile g for launch round `next` (once per round).
__device__ __forceinline__ void enqueue(const WorkList& wl, int g, int next)
{
    if (atomicMax(&wl.listed[g], next) < next) {
        const int pos = atomicAdd(&wl.count[next % 3], 1);
        wl.list[(next & 1) * wl.cap + pos] = g;
    }
}

template <int TH, int TW, int K, int NT, int VAR, typename E>
__device__ __forceinline__ int round_tile(const ImgDev* __restrict__ imgs, ImgCnt* cnt,
                          const int32_t* __restrict__ tile_img, int32_t* tile_state, int g,
                          int round, int ntiles, uint32_t* hist_bits, int32_t* hist_round,
                          typename TileOf<TH, TW, K, NT, VAR, E>::Elem* s_img, uint8_t* s_dirty,
                          uint32_t* s_bits, uint32_t* s_cw, const DecEntry* __restrict__ lut_g,
                          DecEntry* s_lut, int& lut_adj, int* s_count, int* s_last,
                          int* s_exam, const WorkList& wl, int kflags)
{
    using T = TileOf<TH, TW, K, NT, VAR, E>;
    const int tid = threadIdx.x;
    const int ii = (kflags & kOneImage) ? 0 : tile_img[g];
    const ImgDev* d = imgs + ii;
    // A tile that is not this launch's returns at once; the barrier keeps the
    // block's tile hand-out (written by thread 0 before the tile, read by all
    // after it) ordered as a visited tile's barriers do.  Every condition
    // here is the same for the whole block.
    if (((kflags & kOnlyU8) && d->dtype != 1) || ((kflags & kOnlyU16) && d->dtype != 2)) {
        __syncthreads();
        return 0;
    }
    const int r = round - d->round0;
    if (r < 0) {
        __syncthreads();
        return 0;
    }
    const int t0 = r * K;
    const int nsteps = min(K, d->max_steps - t0);
    if (nsteps <= 0) {
        __syncthreads();
        return 0;
    }
    const int lt = g - d->tile0;
    const int ty = lt / d->tiles_x, tx = lt - ty * d->tiles_x;
    const int slot = d->slot;
    // this tile's state pair
    int32_t* st = tile_state + 2 * ((kflags & kStateIsTile) ? (int64_t)g : d->state0 + lt);

    // tile_state[2g] is the latest round for which a tile of g's 3x3 tile
    // neighbourhood asked g to be active (it lowered something during the
    // last 4 steps of the round before); tile_state[2g + 1] is the last round
    // in which g itself lowered something.  Neighbours of this round may raise
    // tile_state[2g] to r + 1 while it is read here (only adding work), so one
    // thread decides and the barrier broadcasts a block-uniform answer.  The
    // tile is staged (and the residency's set-up started) before the answer
    // is known, so its loads overlap the state read; the barrier also
    // completes the staging and orders it after the previous tile's readers
    // of LDS.
    int act = 0, chg = 0;
    if (tid == 0) {
        act = __hip_atomic_load(&st[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        chg = __hip_atomic_load(&st[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const void* src = round_src(d, r);
    void* dst = round_dst(d, r);
    const int gy0 = ty * TH, gx0 = tx * TW;
    const View v = view_of(d);
    if (d->adj != lut_adj) {
        // The block's table follows the image's pairing; the previous tile's
        // readers are past its last barrier, and the decision barrier below
        // orders these writes before this tile's steps.
        lut_adj = d->adj;
        for (int i = tid; i < 256; i += NT) s_lut[i] = lut_g[lut_adj * 256 + i];
    }
    Seed sd{};
    const int64_t words = var_seeded(VAR) ? (int64_t)ntiles * TH * T::WPR : 0;
    sd.prev_bits = hist_bits + ((r + 1) & 1) * words;
    sd.prev_round = hist_round + ((r + 1) & 1) * ntiles;
    sd.cur_bits = hist_bits + (r & 1) * words;
    sd.cur_round = hist_round + (r & 1) * ntiles;
    sd.r = r;
    sd.tile0 = d->tile0;
    sd.tiles_x = d->tiles_x;
    sd.tiles_y = d->tiles_y;
    sd.ty = ty;
    sd.tx = tx;
    sd.g = g;
    T::stage(v, gy0, gx0, src, dst, s_img, tid);
    T::prefetch(v, gy0, gx0, var_seeded(VAR) ? &sd : nullptr, s_dirty, s_cw, tid);
    const int vote = tid == 0 ? ((r == 0 || act >= r) ? 1 : (chg == r - 1 ? 2 : 0)) : 0;
    const int decision = __syncthreads_or(vote == 1) ? 1 : (__syncthreads_or(vote == 2) ? 2 : 0);
    if (decision != 1) {
        // Stable for this round.  The output buffer already equals the input
        // unless the tile changed during the previous round.
        if (decision == 2) {
            T::store(v, gy0, gx0, src, dst, s_img, tid);
            __syncthreads();  // the next tile's staging overwrites s_img
        }
        return 0;
    }
    int last_tau;
    const int count = T::run(v, gy0, gx0, t0, nsteps, src, dst, s_img, s_dirty, s_bits, s_cw,
                             var_seeded(VAR) ? &sd : nullptr, s_lut, s_count, s_last, s_exam,
                             tid, last_tau);
    // Counters and the tiles the next round must visit, from the lanes of
    // wave 0 in parallel (one lane per tile of the 3x3 tile block), so the
    // block's next tile is not held up by a chain of dependent atomics.
    if (tid < 64) {
        if (tid == 0) {
            atomicAdd(&cnt[slot].tile_rounds, 1ull);
            atomicAdd(&cnt[slot].examinations, (unsigned long long)*s_exam);
            if (last_tau >= 0) {
                __hip_atomic_store(&st[1], r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                atomicAdd(&cnt[slot].lowerings, (unsigned long long)count);
                atomicMax(&cnt[slot].last_step, t0 + last_tau);
            }
        }
        // Lowered during the last 4 steps: the tile and those of its 8
        // neighbours within reach must run the next round.  Only pixels next
        // to a pixel lowered during the last 4 steps can be pending, and a
        // change travels at most one pixel per step, so in the next K steps
        // a neighbour's interior can change only if one of those lowerings
        // lies within K of it; a tile none of whose 3x3 tile block is within
        // reach cannot change (K <= tile side).  The seeded variants know
        // where those lowerings are (their change bitmap): wave 0 takes the
        // bounding box and spares the neighbours beyond K + 1 (one pixel of
        // margin); the others ask the whole 3x3 block.  Lowered earlier: the
        // tile itself is visited again (to copy itself across the ping-pong
        // pair).
        if (last_tau >= nsteps - 4) {
            uint32_t ask = 0x1FFu;  // bit 3 (dy + 1) + (dx + 1)
            if constexpr (var_seeded(VAR)) {
                if (nsteps >= 4) {
                    const uint32_t* bits = T::changed(s_dirty, s_bits);
                    int rmin = TH, rmax = -1, cmin = TW, cmax = -1;
                    for (int i = tid; i < TH * T::WPR; i += 64) {
                        const uint32_t w = bits[i];
                        if (!w) continue;
                        const int row = i / T::WPR, c0 = 32 * (i - row * T::WPR);
                        rmin = min(rmin, row);
                        rmax = max(rmax, row);
                        cmin = min(cmin, c0 + __ffs(w) - 1);
                        cmax = max(cmax, c0 + 31 - __clz(w));
                    }
#pragma unroll
                    for (int o = 32; o >= 1; o >>= 1) {
                        rmin = min(rmin, __shfl_xor(rmin, o));
                        rmax = max(rmax, __shfl_xor(rmax, o));
                        cmin = min(cmin, __shfl_xor(cmin, o));
                        cmax = max(cmax, __shfl_xor(cmax, o));
                    }
                    if (rmax >= 0) {
                        constexpr int REACH = K + 1;
                        const bool up = rmin <= REACH, down = rmax >= TH - 1 - REACH;
                        const bool left = cmin <= REACH, right = cmax >= TW - 1 - REACH;
                        const uint32_t rows = (up ? 1u : 0u) | 2u | (down ? 4u : 0u);
                        const uint32_t cols = (left ? 1u : 0u) | 2u | (right ? 4u : 0u);
                        ask = 0u;
#pragma unroll
                        for (int q = 0; q < 9; ++q)
                            if (((rows >> (q / 3)) & 1u) && ((cols >> (q % 3)) & 1u)) ask |= 1u << q;
                    }
                }
            }
            if (tid < 9 && ((ask >> tid) & 1u)) {
                const int y = ty + tid / 3 - 1, x = tx + tid % 3 - 1;
                if (y >= 0 && y < d->tiles_y && x >= 0 && x < d->tiles_x) {
                    __hip_atomic_fetch_max(&tile_state[2 * (d->state0 + y * d->tiles_x + x)],
                                           r + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (wl.list != nullptr) enqueue(wl, d->tile0 + y * d->tiles_x + x, round + 1);
                }
            }
        } else if (last_tau >= 0 && tid == 0 && wl.list != nullptr) {
            enqueue(wl, g, round + 1);
        }
    }
    return 1;
}

template <int TH, int TW, int K, int NT, int VAR, typename E>
__global__ __attribute__((amdgpu_flat_work_group_size(1, NT),
                          amdgpu_waves_per_eu(lds_waves_per_eu<TileOf<TH, TW, K, NT, VAR, E>, NT, TH, VAR>())))
void k_round(const ImgDev* __restrict__ imgs, ImgCnt* cnt,
                                              const int32_t* __restrict__ tile_img,
                                              int32_t* tile_last, int ntiles, int round,
                                              const DecEntry* __restrict__ lut_g,
                                              uint32_t* hist_bits, int32_t* hist_round,
                                              WorkList wl, const int32_t* round_base,
                                              int kflags)
{
    using T = TileOf<TH, TW, K, NT, VAR, E>;
    if (round_base != nullptr) round += *round_base;
    __shared__ __align__(16) typename T::Elem s_img[T::IMG_ELEMS];
    __shared__ __align__(16) uint8_t s_dirty[T::DIRTY_ELEMS];
    __shared__ uint32_t s_bits[T::BITS_WORDS];
    __shared__ uint32_t s_cw[T::CW_WORDS];
    __shared__ DecEntry s_lut[256];
    __shared__ int s_count, s_last, s_exam;
    int lut_adj = -1;
    const bool all = wl.list == nullptr || round == wl.full;
    const int n = all ? ntiles : wl.count[round % 3];
    if (wl.list != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {
        wl.count[(round + 2) % 3] = 0;
        wl.grab[2 * ((round + 2) % 3)] = 0;
        wl.grab[2 * ((round + 2) % 3) + 1] = 0;
    }
    const int32_t* mine = all ? nullptr : wl.list + (round & 1) * wl.cap;
    // Each block takes its first tile by its index and every later one from
    // a counter shared by the round's blocks, so blocks that drew cheap
    // tiles take more of them (tiles differ widely in cost: partial tiles
    // at image borders, quiet ones that are skipped).  Thread 0 claims the
    // next position while the current tile runs; two slots, so that a slot
    // is written again only after every thread has passed a barrier of the
    // tile in between.  The u8 and u16 launches of one round draw from
    // counters of their own.
    __shared__ int s_next[2];
    int32_t* grab = wl.list != nullptr ? wl.grab + 2 * (round % 3) + ((kflags & kOnlyU16) ? 1 : 0)
                                       : nullptr;
    int i = blockIdx.x;
    for (int k = 0; i < n; ++k) {
        if (threadIdx.x == 0)
            s_next[k & 1] = grab ? (int)gridDim.x + atomicAdd(grab, 1) : i + (int)gridDim.x;
        round_tile<TH, TW, K, NT, VAR, E>(imgs, cnt, tile_img, tile_last, all ? i : mine[i], round,
                                          ntiles, hist_bits, hist_round, s_img, s_dirty, s_bits,
                                          s_cw, lut_g, s_lut, lut_adj, &s_count, &s_last, &s_exam,
                                          wl, kflags);
        i = s_next[k & 1];
    }
}

// ------------------------------------------------------------------ k_coop
//
// All rounds in one cooperative launch (every block resident): each round
// processes the tile list like k_round, then the whole grid synchronises.
// active[round % 3] counts the tiles processed in a round; a round in which
// no tile was active means every image is stable (a tile is skipped only when
// its neighbourhood was quiet for the last 4 steps), so all blocks leave
// together.  The counter of round r is read by every block right after the
// grid barrier of round r and is cleared during round r + 2, after the next
// barrier has proved those reads complete.

template <int TH, int TW, int K, int NT, int VAR, typename E>
__global__ __attribute__((amdgpu_flat_work_group_size(1, NT),
                          amdgpu_waves_per_eu(lds_waves_per_eu<TileOf<TH, TW, K, NT, VAR, E>, NT, TH, VAR>())))
void k_coop(const ImgDev* __restrict__ imgs, ImgCnt* cnt,
                                             const int32_t* __restrict__ tile_img,
                                             int32_t* tile_last, int ntiles,
                                             const DecEntry* __restrict__ lut_g, int32_t* active,
                                             int32_t* rounds_out, int max_rounds,
                                             uint32_t* hist_bits, int32_t* hist_round, int kflags)
{
    using T = TileOf<TH, TW, K, NT, VAR, E>;
    __shared__ __align__(16) typename T::Elem s_img[T::IMG_ELEMS];
    __shared__ __align__(16) uint8_t s_dirty[T::DIRTY_ELEMS];
    __shared__ uint32_t s_bits[T::BITS_WORDS];
    __shared__ uint32_t s_cw[T::CW_WORDS];
    __shared__ DecEntry s_lut[256];
    __shared__ int s_count, s_last, s_exam;
    const int tid = threadIdx.x;
    int lut_adj = -1;
    cooperative_groups::grid_group grid = cooperative_groups::this_grid();
    int round = 0;
    for (;; ++round) {
        if (blockIdx.x == 0 && tid == 0)
            __hip_atomic_store(&active[(round + 1) % 3], 0, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        int mine = 0;
        for (int g = blockIdx.x; g < ntiles; g += gridDim.x)
            mine += round_tile<TH, TW, K, NT, VAR, E>(imgs, cnt, tile_img, tile_last, g, round,
                                                 ntiles, hist_bits, hist_round, s_img, s_dirty,
                                                 s_bits, s_cw, lut_g, s_lut, lut_adj, &s_count,
                                                 &s_last, &s_exam, WorkList{}, kflags);
        if (tid == 0 && mine) atomicAdd(&active[round % 3], mine);
        // Stores of every wave must be acknowledged before the grid barrier
        // publishes them.
        __builtin_amdgcn_s_waitcnt(0);
        grid.sync();
        const int a = __hip_atomic_load(&active[round % 3], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
        if (a == 0 || round + 1 >= max_rounds) break;
    }
    if (blockIdx.x == 0 && tid == 0) *rounds_out = round + 1;
}

// ------------------------------------------------------------------ k_flow
//
// Small images: the whole run in one launch, every tile of an
// image held by a block of its own from its first step to its last, windows
// in registers and region in LDS.  Nothing is staged between rounds: after K
// steps a block publishes its interior cells and takes its halo cells from
// the tiles around it, and neighbours wait for each other only.
//
// A round of launches costs about 7500 cycles between launches, 6000 to stage
// a tile and 4000 to set it up and store it, beside some 20000 for 16 steps
// (512x512 ridges, 140 rounds: 2.16 ms).  Here an exchange costs about 4000
// (one trip to memory and back, the region's windows compared), which lets a
// round have 8 steps and a region two thirds the size: 12000 cycles a round,
// 1.37 ms.  What bounds it now is the steps' chain of latencies (930 cycles a
// step, two thirds of them the vector instructions of the busiest tile's
// waves, few lanes of which are active).
//
// Exchange.  A cell (2x2 pixels) travels as 64-bit words whose high half is
// the round's tag, so a word that carries the tag carries the data and no
// second flag or fence is needed: u8 cells one word, u16 cells two (one per
// pixel row).  Words are stored and polled with relaxed agent-scope atomics
// (the XCDs' L2 caches are not coherent with each other).  Two copies
// alternate by round parity: a tile overwrites its round r words in round
// r + 2, which it enters only after every neighbour's round r + 1 words
// arrived, and a neighbour publishes those after a barrier behind its reads
// of round r.
//
// Candidates.  A candidate not pending was examined at the values its 3x3
// holds now and not lowered; the decision is a function of the 3x3, so this
// holds in the halo too, where the values of the last steps were not exact:
// after the exchange each window is compared with the region's new values and
// every candidate next to a difference becomes pending.
//
// Convergence.  After every vote_every-th round a tile adds one to that round's
// votes, and one in the high half when it lowered an interior pixel during
// the round's last 4 steps (one word, so that neither is seen without the
// other).  The first tile reads one vote word a round; when all tiles have
// voted and none was active it marks the image stable (ImgCnt.pad): every
// tile's interior is then final, and its block stores it and takes the next
// tile.  (All blocks reading the word that all blocks add to costs tens of
// thousands of cycles a round.)  Tiles of one image are never further apart
// in rounds than in tiles (at most kFlowMaxSide), so a ring of kFlowRing vote
// words is enough; the first tile clears each half a ring after its use.
//
// Progress.  Blocks take tiles in order.  Every image before the oldest
// unfinished one is finished, so its blocks come back for tiles; the oldest
// unfinished one has at most gridDim.x tiles and all blocks become resident
// (the grid is no larger than the device holds, other kernels end, and the
// host lets this process's waiting kernels run together only where all fit),
// so all its tiles get a block and none waits for a tile without one.  Every
// wait and the number of rounds (kFlowMaxRounds) are bounded all the same: a block that runs
// out marks its image given up, sets the abort word and leaves, as do all that
// see either, and the host runs the images that are not stable on the rounds
// of launches.  An image's mark changes once (compare and swap), and its tiles
// are stored when it says stable only, so images given up are untouched.

__device__ __forceinline__ uint64_t flow_load(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t flow_load(const int32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void flow_store(uint64_t* p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void flow_store(int32_t* p, int32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waves per SIMD the compiler fits k_flow's registers to: two blocks to a
// compute unit for the 48x48 tiles (they serve the images that need them
// all), else what one block of 16 waves takes.
constexpr int flow_waves_per_eu(int nt, int th) { return nt == 1024 && th == 48 ? 8 : 4; }

// Marks an image unless it already has a mark; the mark it has.
__device__ __forceinline__ int flow_mark(int32_t* at, int mark)
{
    const int was = atomicCAS(at, kFlowRunning, mark);
    return __builtin_amdgcn_readfirstlane(was == kFlowRunning ? mark : was);
}

template <int TH, int TW, int K, int NT>
__global__ __launch_bounds__(NT, flow_waves_per_eu(NT, TH)) void k_flow(const FlowImg* __restrict__ imgs,
                                             const int32_t* __restrict__ tile_img, int ntiles,
                                             ImgCnt* cnt, const DecEntry* __restrict__ lut_g,
                                             int32_t* ctl, uint64_t* exch, int max_polls,
                                             int max_rounds, int vote_every)
{
    using T = RTile<TH, TW, K, NT, false>;
    constexpr int PPT = T::PPT, RWP = T::RWP;
    __shared__ __align__(16) uint16_t s_img[T::IMG_ELEMS];
    __shared__ __align__(16) uint8_t s_flags[T::DIRTY_ELEMS];
    __shared__ DecEntry s_lut[256];
    __shared__ int s_tile, s_act, s_mark, s_count, s_last;
    __shared__ unsigned long long s_exam;
    const int tid = threadIdx.x;
    int lut_adj = -1;
    const int vote_shift = 31 - __clz(vote_every);
    for (;;) {
        if (tid == 0) s_tile = flow_load(&ctl[kFlowAbort]) ? ntiles : atomicAdd(&ctl[kFlowNext], 1);
        __syncthreads();
        const int g = s_tile;
        if (g >= ntiles) break;
        const FlowImg im = imgs[tile_img != nullptr ? tile_img[g] : 0];
        const int lt = g - im.tile0, ty = lt / im.tiles_x, tx = lt - ty * im.tiles_x;
        const int gy0 = ty * TH, gx0 = tx * TW;
        View d;
        d.pitch = im.pitch;
        d.h = im.h;
        d.w = im.w;
        d.dtype = im.dtype;
        d.lambda = im.lambda;
        if (im.adj != lut_adj) {
            lut_adj = im.adj;
            for (int i = tid; i < 256; i += NT) s_lut[i] = lut_g[lut_adj * 256 + i];
        }
        if (tid == 0) {
            s_act = 0;
            s_mark = kFlowRunning;
            s_count = 0;
            s_last = -1;
            s_exam = 0ull;
        }
        if (tid < T::DIRTY_ELEMS / 4) reinterpret_cast<uint32_t*>(s_flags)[tid] = 0u;
        T::stage_once(d, gy0, gx0, im.image, s_img, tid);
        __syncthreads();
        typename T::Cells q;
        T::open(q, d, gy0, gx0, s_img, tid);
        // this thread's cells in the exchange: word index, or none (outside
        // the image), and whether the tile owns them
        const int cells_y = (im.h + 1) / 2, cells_x = (im.w + 1) / 2;
        const int64_t ncells = (int64_t)cells_y * cells_x;
        const int wpc = im.dtype == 1 ? 1 : 2;  // words per cell
        int word[PPT];
        bool own[PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            int a, b;
            const bool valid = T::cell(tid, k, a, b);
            const int ga = (gy0 - K) / 2 + a, gb = (gx0 - K) / 2 + b;
            const bool live = valid && ga >= 0 && ga < cells_y && gb >= 0 && gb < cells_x;
            own[k] = live && a >= K / 2 && a < K / 2 + TH / 2 && b >= K / 2 && b < K / 2 + TW / 2;
            word[k] = live ? wpc * (ga * cells_x + gb) : -1;
        }
        __syncthreads();  // every window is read

        uint64_t* const ex = exch + im.word0;
        const Lambda lambda = lambda_of(im.lambda);
        int lowered = 0, last = -1;  // of the wave, over all rounds
        // (a candidate is examined once, and again after a pixel of its 4x4 window
        // fell: 768 candidates of a wave times 16 pixels of 65535 levels fit 32
        // bits)
        unsigned exams = 0;
        int32_t* const image_mark = &cnt[im.slot].pad;
        int32_t* const ring = ctl + im.ctl0;
        const bool counts = lt == 0 && tid < 64;  // the wave that counts the image's votes
        int vote = 0;                             // the next vote to count
        int end = kFlowRunning;
        int r = 0;
        for (;; ++r) {
            typename T::Counts n;
            T::steps(q, s_img, s_flags, nullptr, K, tid, s_lut, lambda, n);
            lowered += n.lowered;
            exams += n.exams;
            if (n.last >= 0) last = r * K + n.last;
            if (n.last >= K - 4 && (tid & 63) == 0) s_act = 1;
            const uint32_t tag = (uint32_t)r + 1u;
            uint64_t* const slot = ex + (int64_t)(tag & 1) * wpc * ncells;
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                if (!own[k]) continue;
                // the cell's pixel rows: window columns 1 and 2 of rows 1 and 2
                const uint32_t r0 = __builtin_amdgcn_alignbyte(q.win[k][3], q.win[k][2], 2);
                const uint32_t r1 = __builtin_amdgcn_alignbyte(q.win[k][5], q.win[k][4], 2);
                if (wpc == 1) {
                    flow_store(&slot[word[k]],
                               (uint64_t)tag << 32 | __builtin_amdgcn_perm(r1, r0, 0x06040200u));
                } else {
                    flow_store(&slot[word[k]], (uint64_t)tag << 32 | r0);
                    flow_store(&slot[word[k] + 1], (uint64_t)tag << 32 | r1);
                }
            }
            lds_barrier();  // s_act complete; every read of this round's flags done
            if (tid == 0) {
                if ((r & (vote_every - 1)) == vote_every - 1) {
                    const int v = r >> vote_shift;
                    (void)__hip_atomic_fetch_add(&ring[v & (kFlowRing - 1)], 1 + (s_act << 16),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    // the word used half a ring ago: every tile is past it
                    // and none is back at it
                    if (lt == 0 && v >= kFlowRing / 2)
                        flow_store(&ring[(v + kFlowRing / 2) & (kFlowRing - 1)], 0);
                }
                s_act = 0;
            }
            if (tid < T::DIRTY_ELEMS / 4) reinterpret_cast<uint32_t*>(s_flags)[tid] = 0u;
            // halo cells of this round
            uint64_t got[PPT][2];
            int mark = kFlowRunning;
            for (int polls = 0;; ++polls) {
                // (every load goes out before the first is waited for; the
                // words all blocks share are read as seldom as will do)
                int32_t m = kFlowRunning, votes = 0;
                if (polls == 0 ? tid < 64 : (polls & 3) == 3) m = flow_load(image_mark);
                if (counts && polls == 0 && (vote + 1) << vote_shift <= r)
                    votes = flow_load(&ring[vote & (kFlowRing - 1)]);
#pragma unroll
                for (int k = 0; k < PPT; ++k) {
                    if (word[k] < 0 || own[k]) continue;
                    got[k][0] = flow_load(&slot[word[k]]);
                    got[k][1] = flow_load(&slot[word[k] + wpc - 1]);
                }
                mark = __builtin_amdgcn_readfirstlane(m);
                if (counts) {
                    votes = __builtin_amdgcn_readfirstlane(votes);
                    if ((votes & 0xFFFF) == im.tiles_x * im.tiles_y) {
                        // every tile is through that round
                        if (votes >> 16 == 0 && mark == kFlowRunning)
                            mark = flow_mark(image_mark, kFlowStable);
                        vote = max(vote + 1, (r >> vote_shift) - 1);
                    }
                }
                bool wait = false;
#pragma unroll
                for (int k = 0; k < PPT; ++k) {
                    if (word[k] < 0 || own[k]) continue;
                    wait |= (uint32_t)(got[k][0] >> 32) != tag || (uint32_t)(got[k][1] >> 32) != tag;
                }
                if (__ballot(wait) == 0 || mark != kFlowRunning) break;
                if (polls >= max_polls ||
                    ((polls & 15) == 15 &&
                     __builtin_amdgcn_readfirstlane(flow_load(&ctl[kFlowAbort])) != 0)) {
                    mark = flow_mark(image_mark, kFlowGivenUp);
                    break;
                }
                if (polls > 8) __builtin_amdgcn_s_sleep(1);
            }
            if (mark == kFlowRunning && r + 1 >= max_rounds) mark = flow_mark(image_mark, kFlowGivenUp);
            if (mark != kFlowRunning && (tid & 63) == 0) s_mark = mark;
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                if (word[k] < 0 || own[k]) continue;
                const uint32_t v = (uint32_t)got[k][0];
                const uint32_t r0 = wpc == 1 ? (v & 0xFFu) | (v & 0xFF00u) << 8 : v;
                const uint32_t r1 = wpc == 1 ? (v >> 16 & 0xFFu) | (v >> 24) << 16 : (uint32_t)got[k][1];
                uint16_t* p = s_img + 2 * q.base[k] + RWP + 1;
                p[0] = (uint16_t)r0;
                p[1] = (uint16_t)(r0 >> 16);
                p[RWP] = (uint16_t)r1;
                p[RWP + 1] = (uint16_t)(r1 >> 16);
            }
            lds_barrier();
            end = s_mark;
            if (end != kFlowRunning) break;
            T::refresh(q, s_img);
            lds_barrier();  // windows are read before the next step writes
        }
        if (end != kFlowStable) {
            if (tid == 0) flow_store(&ctl[kFlowAbort], 1);
            break;
        }
        T::store(d, gy0, gx0, im.image, im.image, s_img, tid);
        if ((tid & 63) == 0) {
            if (lowered) {
                atomicAdd(&s_count, lowered);
                atomicMax(&s_last, last);
            }
            if (exams) atomicAdd(&s_exam, (unsigned long long)exams);
        }
        __syncthreads();
        if (tid == 0) {
            ImgCnt* c = cnt + im.slot;
            atomicAdd(&c->tile_rounds, (unsigned long long)(r + 1));
            atomicAdd(&c->examinations, s_exam);
            if (s_count) {
                atomicAdd(&c->lowerings, (unsigned long long)(uint32_t)s_count);
                atomicMax(&c->last_step, s_last);
            }
        }
        __syncthreads();  // the next tile resets the block's totals
    }
}

// Clears the control words and the exchange words of a run and, for one image,
// writes its descriptor.
__global__ void k_flow_init(ImgCnt* cnt, int nimg, int32_t* ctl, int nctl, uint4* exch,
                            int64_t nquad, FlowImg* dst, FlowImg one)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = i; k < nquad; k += step) exch[k] = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t k = i; k < nctl; k += step) ctl[k] = 0;
    if (i < nimg) {
        cnt[i].lowerings = 0ull;
        cnt[i].tile_rounds = 0ull;
        cnt[i].last_step = -1;
        cnt[i].pad = kFlowRunning;
        cnt[i].examinations = 0ull;
    }
    if (dst != nullptr && i == 0) *dst = one;
}

template <int TH, int TW, int K, int NT, int VAR, typename E>
hipError_t launch_coop_t(hipStream_t stream, const ImgDev* imgs, ImgCnt* cnt,
                         const int32_t* tile_img, int32_t* tile_last, int ntiles,
                         const DecEntry* lut, int32_t* active, int32_t* rounds_out,
                         int max_rounds, int num_cus, uint32_t* hist_bits, int32_t* hist_round,
                         int kflags)
{
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void*>(&k_coop<TH, TW, K, NT, VAR, E>), NT, 0);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    const int grid = max(1, min(ntiles, per_cu * num_cus));
    void* args[] = {(void*)&imgs,       (void*)&cnt,       (void*)&tile_img,
                    (void*)&tile_last,  (void*)&ntiles,    (void*)&lut,
                    (void*)&active,     (void*)&rounds_out, (void*)&max_rounds,
                    (void*)&hist_bits,  (void*)&hist_round, (void*)&kflags};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&k_coop<TH, TW, K, NT, VAR, E>),
                                      dim3(grid), dim3(NT), args, 0, stream);
}

template <int TH, int TW, int K, int NT, int VAR, typename E>
hipError_t launch_round_t(hipStream_t stream, const ImgDev* imgs, ImgCnt* cnt,
                          const int32_t* tile_img, int32_t* tile_last, int ntiles, int round,
                          const DecEntry* lut, int num_cus, uint32_t* hist_bits,
                          int32_t* hist_round, WorkList wl, const int32_t* round_base, int kflags)
{
    // As many blocks as fit on the device at once (registers, LDS and thread
    // slots of this instantiation), each looping over the tiles.
    static int per_cu = 0;
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &n, reinterpret_cast<const void*>(&k_round<TH, TW, K, NT, VAR, E>), NT, 0) !=
                hipSuccess ||
            n < 1)
            n = 1;
        per_cu = n;
    }
    const int grid = max(1, min(ntiles, per_cu * num_cus));
    hipLaunchKernelGGL((k_round<TH, TW, K, NT, VAR, E>), dim3(grid), dim3(NT), 0, stream, imgs, cnt,
                       tile_img, tile_last, ntiles, round, lut, hist_bits, hist_round, wl,
                       round_base, kflags);
    return hipGetLastError();
}

// -------------------------------------------------------------- k_worklist
//
// The re-examination rule of section 2.2 as explicit per-class candidate
// lists.  A candidate is pending when a pixel of its 3x3 (itself included)
// was lowered since its last examination; the visit of its class examines
// every pending candidate of that class once and clears it; a lowered pixel
// marks its 3x3 pending (one bit per lattice cell and class, set with an
// atomic so each cell enters its class's list once).  The class being
// visited receives no marks from its own step except the lowered pixels
// themselves, which become the next list of that class.  Started with every
// interior candidate pending, the engine examines exactly the candidates
// the sequential dirty-pixel sweep examines.
//
// Lists hold (lattice row << 16) | lattice column and live in LDS; a list
// that overflows is dropped and its class's next visit scans the bitmap
// instead (the bitmap is always exact).  The pending bitmaps stay in LDS when
// they fit, else in global memory.  One block of kWlThreads threads per image;
// two barriers per step.

// Pending-bitmap access of k_worklist.  In global memory the words are read
// and written with device-scope atomics, which go to L2 like the bit-setting
// atomics, so no wave reads a stale copy from its CU's L1.
template <bool GBITS>
__device__ __forceinline__ uint32_t wl_load(uint32_t* w)
{
    if constexpr (GBITS) return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *w;
}
template <bool GBITS>
__device__ __forceinline__ void wl_store(uint32_t* w, uint32_t v)
{
    if constexpr (GBITS) __hip_atomic_store(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *w = v;
}
template <bool GBITS>
__device__ __forceinline__ uint32_t wl_or(uint32_t* w, uint32_t m)
{
    if constexpr (GBITS) return __hip_atomic_fetch_or(w, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return atomicOr(w, m);
}
template <bool GBITS>
__device__ __forceinline__ void wl_and(uint32_t* w, uint32_t m)
{
    if constexpr (GBITS) __hip_atomic_fetch_and(w, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else atomicAnd(w, m);
}

template <typename E, bool GBITS>
__global__ __launch_bounds__(kWlThreads) void k_worklist(const WlImg* __restrict__ imgs,
                                                       ImgCnt* cnt,
                                                       const DecEntry* __restrict__ lut_g,
                                                       int32_t* steps_out)
{
    __shared__ DecEntry s_lut[256];
    __shared__ uint32_t s_lbits[GBITS ? 1 : kWlLdsWords];
    __shared__ uint32_t s_list[5][kWlListCap];
    __shared__ int s_n[5], s_ovf[5], s_map[4];
    __shared__ int s_j, s_low, s_quiet, s_step, s_last;
    __shared__ unsigned long long s_exam, s_lowsum;
    const int tid = threadIdx.x;
    const WlImg im = imgs[blockIdx.x];
    E* img = static_cast<E*>(im.image);
    const int64_t P = im.pitch;
    const int H = im.h, W = im.w;
    const int LH = (H + 1) / 2, LW = (W + 1) / 2, LWW = (LW + 31) / 32, CW = LH * LWW;
    uint32_t* bits = GBITS ? im.gbits : s_lbits;
    for (int i = tid; i < 256; i += kWlThreads) s_lut[i] = lut_g[im.adj * 256 + i];
    if (tid < 5) {
        s_n[tid] = 0;
        s_ovf[tid] = 1;   // first visit of each class scans its bitmap
    }
    if (tid < 4) s_map[tid] = tid;
    if (tid == 0) {
        s_j = 4;
        s_low = 0;
        s_quiet = 0;
        s_step = im.step0;
        s_last = -1;
        s_exam = 0ull;
        s_lowsum = 0ull;
    }
    // Initial pending sets.  Cell (a, b) of class (si, sj) is pixel
    // (2a + si, 2b + sj); only interior pixels are ever pending.  With init 1
    // a candidate is pending when a pixel of its 3x3 differs from the state
    // one tiled round earlier: a pixel-change bitmap (1 bit per pixel, rows of
    // DW words) is built first, in the list storage while it is unused when
    // it fits there.
    const int DW = (W + 31) / 32;
    uint32_t* dmap = &s_list[0][0];
    const bool dfast = im.init == 1 && H * DW <= 5 * kWlListCap;
    if (dfast) {
        const E* prev = static_cast<const E*>(im.prev);
        for (int wd = tid; wd < H * DW; wd += kWlThreads) {
            const int y = wd / DW, x0 = 32 * (wd - y * DW);
            const E* ra = img + (int64_t)y * P + x0;
            const E* rb = prev + (int64_t)y * P + x0;
            const int nx = min(32, W - x0);
            uint32_t m = 0u;
            for (int t = 0; t < nx; ++t) m |= (uint32_t)(ra[t] != rb[t]) << t;
            dmap[wd] = m;
        }
        __syncthreads();
    }
    for (int wd = tid; wd < 4 * CW; wd += kWlThreads) {
        const int c = wd / CW, rem = wd - c * CW;
        const int a = rem / LWW, j0 = 32 * (rem - a * LWW);
        const int i = 2 * a + (c >> 1);
        uint32_t word = 0u;
        if (i >= 1 && i <= H - 2) {
            for (int t = 0; t < 32; ++t) {
                const int j = 2 * (j0 + t) + (c & 1);
                if (j < 1 || j > W - 2) continue;
                bool pend = true;
                if (dfast) {
                    pend = false;
                    for (int di = -1; di <= 1; ++di) {
                        const uint32_t* row = dmap + (i + di) * DW;
                        for (int dj = -1; dj <= 1; ++dj) {
                            const int x = j + dj;
                            pend |= ((row[x >> 5] >> (x & 31)) & 1u) != 0u;
                        }
                    }
                } else if (im.init == 1) {
                    const E* prev = static_cast<const E*>(im.prev);
                    pend = false;
                    for (int di = -1; di <= 1 && !pend; ++di)
                        for (int dj = -1; dj <= 1; ++dj) {
                            const int64_t o = (int64_t)(i + di) * P + (j + dj);
                            if (img[o] != prev[o]) {
                                pend = true;
                                break;
                            }
                        }
                }
                if (pend) word |= 1u << t;
            }
        }
        wl_store<GBITS>(&bits[wd], word);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    const Lambda lambda = lambda_of(im.lambda);
    unsigned long long my_exam = 0ull;
    for (;;) {
        const int t = s_step;
        if (s_quiet >= 4 || t >= im.max_steps) break;
        const int c = t & 3, si = c >> 1, sj = c & 1;
        const int L = s_map[c], J = s_j;
        const bool scan = s_ovf[L] != 0;
        const int n = scan ? CW : min(s_n[L], kWlListCap);
        int my_low = 0;
        // one candidate (or, scanning, one bitmap word) per iteration
        for (int k = tid; k < n; k += kWlThreads) {
            uint32_t cells, wbase;
            int a, b0;
            if (scan) {
                cells = wl_load<GBITS>(&bits[c * CW + k]);
                if (!cells) continue;
                wl_store<GBITS>(&bits[c * CW + k], 0u);   // no other thread touches it this step
                a = k / LWW;
                b0 = 32 * (k - a * LWW);
                wbase = c * CW + k;
            } else {
                const uint32_t e = s_list[L][k];
                a = (int)(e >> 16);
                const int b = (int)(e & 0xFFFFu);
                b0 = b & ~31;
                cells = 1u << (b & 31);
                wbase = c * CW + a * LWW + (b >> 5);
                wl_and<GBITS>(&bits[wbase], ~cells);
            }
            uint32_t relower = 0u;
            while (cells) {
                const int bit = __ffs(cells) - 1;
                cells &= cells - 1u;
                ++my_exam;
                const int i = 2 * a + si, j = 2 * (b0 + bit) + sj;
                E* p = img + (int64_t)i * P + j;
                const uint32_t v = p[0];
                const uint32_t nbv[8] = {p[1], p[-P + 1], p[-P], p[-P - 1],
                                         p[-1], p[P - 1], p[P], p[P + 1]};
                uint32_t alpha;
                if (!decide(ring_of(v, nbv), s_lut, lambda, alpha)) continue;
                p[0] = (E)alpha;
                ++my_low;
                relower |= 1u << bit;
                // itself: the next list of this class
                const int pos = atomicAdd(&s_n[J], 1);
                if (pos < kWlListCap) s_list[J][pos] = ((uint32_t)a << 16) | (uint32_t)(b0 + bit);
                else s_ovf[J] = 1;
                // its 8 neighbours (other classes), interior only
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int di = q < 3 ? -1 : (q < 5 ? 0 : 1);
                    const int dj = q < 3 ? q - 1 : (q == 3 ? -1 : (q == 4 ? 1 : q - 6));
                    const int y = i + di, x = j + dj;
                    if (y < 1 || y > H - 2 || x < 1 || x > W - 2) continue;
                    const int cy = ((y & 1) << 1) | (x & 1);
                    const int ay = y >> 1, by = x >> 1;
                    const uint32_t m = 1u << (by & 31);
                    const uint32_t old = wl_or<GBITS>(&bits[cy * CW + ay * LWW + (by >> 5)], m);
                    if (old & m) continue;
                    const int lk = s_map[cy];
                    const int pp = atomicAdd(&s_n[lk], 1);
                    if (pp < kWlListCap) s_list[lk][pp] = ((uint32_t)ay << 16) | (uint32_t)by;
                    else s_ovf[lk] = 1;
                }
            }
            if (relower) {
                // lowered cells are pending again for their next visit
                wl_or<GBITS>(&bits[wbase], relower);
            }
        }
        if (my_low) atomicAdd(&s_low, my_low);
        // The image and (in global memory) the bitmaps are shared through
        // memory: every wave's writes must be complete before the barrier.
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) {
            // the lowered pixels of this step are the next list of class c
            s_map[c] = J;
            s_j = L;
            s_n[L] = 0;
            s_ovf[L] = 0;
            if (s_low) {
                s_quiet = 0;
                s_last = t - im.step0;
                s_lowsum += (unsigned long long)s_low;
            } else {
                ++s_quiet;
            }
            s_low = 0;
            s_step = t + 1;
        }
        __syncthreads();
    }
    if (my_exam) atomicAdd(&s_exam, my_exam);
    __syncthreads();
    if (tid == 0) {
        ImgCnt* ct = cnt + im.slot;
        atomicAdd(&ct->lowerings, s_lowsum);
        atomicAdd(&ct->examinations, s_exam);
        if (s_last >= 0) atomicMax(&ct->last_step, im.step0 + s_last);
        steps_out[blockIdx.x] = s_step;
    }
}

template <int TH, int TW, int K, int NT>
int flow_capacity_t(int num_cus)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void*>(&k_flow<TH, TW, K, NT>), NT, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per_cu * num_cus;
}

template <int TH, int TW, int K, int NT>
hipError_t launch_flow_t(hipStream_t stream, const FlowRun& r)
{
    hipLaunchKernelGGL((k_flow<TH, TW, K, NT>), dim3(r.grid), dim3(NT), 0, stream, r.imgs, r.tile_img,
                       r.ntiles, r.cnt, r.lut, r.ctl, r.exch, r.max_polls, r.max_rounds, r.vote_every);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_init_state(hipStream_t stream, ImgCnt* cnt, int nimg, int32_t* tile_last,
                             int ntiles, int32_t* hist_round, WorkList wl)
{
    const int n = max(max(nimg, 2 * ntiles), 3);
    hipLaunchKernelGGL(k_init_state, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0,
                       stream, cnt, nimg, tile_last, ntiles, hist_round, wl);
    return hipGetLastError();
}

hipError_t launch_serve_init(hipStream_t stream, const ImgDev* imgs, int nimg, ImgCnt* cnt,
                             int32_t* tile_state)
{
    hipLaunchKernelGGL(k_serve_init, dim3(nimg), dim3(kThreads), 0, stream, imgs, cnt, tile_state);
    return hipGetLastError();
}

hipError_t launch_worklist(hipStream_t stream, const WlImg* imgs, int nimg, int dtype,
                           bool gbits, ImgCnt* cnt, const DecEntry* lut, int32_t* steps_out)
{
    if (nimg <= 0) return hipSuccess;
    const dim3 grid(nimg), block(kWlThreads);
    if (dtype == 1) {
        if (gbits) hipLaunchKernelGGL((k_worklist<uint8_t, true>), grid, block, 0, stream, imgs, cnt, lut, steps_out);
        else hipLaunchKernelGGL((k_worklist<uint8_t, false>), grid, block, 0, stream, imgs, cnt, lut, steps_out);
    } else {
        if (gbits) hipLaunchKernelGGL((k_worklist<uint16_t, true>), grid, block, 0, stream, imgs, cnt, lut, steps_out);
        else hipLaunchKernelGGL((k_worklist<uint16_t, false>), grid, block, 0, stream, imgs, cnt, lut, steps_out);
    }
    return hipGetLastError();
}

int flow_capacity(FlowShape s, int num_cus)
{
#define X(a, b, c, n) \
    if (s.th == a && s.tw == b && s.k == c && s.nt == n) return flow_capacity_t<a, b, c, n>(num_cus);
    THIN_FLOW_SHAPES(X)
#undef X
    return 0;
}

hipError_t launch_flow(hipStream_t stream, FlowShape s, const FlowRun& r)
{
#define X(a, b, c, n) \
    if (s.th == a && s.tw == b && s.k == c && s.nt == n) return launch_flow_t<a, b, c, n>(stream, r);
    THIN_FLOW_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_flow_init(hipStream_t stream, const FlowRun& r, int nimg, int nctl,
                            int64_t exch_words, const FlowImg* one)
{
    const int64_t quads = (exch_words + 1) / 2;
    const int64_t want = max(max((int64_t)nimg, (int64_t)nctl), quads);
    const int grid = (int)min((int64_t)1024, (want + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(k_flow_init, dim3(max(grid, (nimg + kThreads - 1) / kThreads)), dim3(kThreads),
                       0, stream, r.cnt, nimg, r.ctl, nctl, reinterpret_cast<uint4*>(r.exch), quads,
                       one ? const_cast<FlowImg*>(r.imgs) : nullptr, one ? *one : FlowImg{});
    return hipGetLastError();
}

hipError_t launch_set_desc(hipStream_t stream, ImgDev* dst, const ImgDev& d)
{
    hipLaunchKernelGGL(k_set_desc, dim3(1), dim3(64), 0, stream, dst, d);
    return hipGetLastError();
}

hipError_t launch_advance(hipStream_t stream, int32_t* round_base, int n)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, stream, round_base, n);
    return hipGetLastError();
}

hipError_t launch_step(hipStream_t stream, const ImgDev* img_host, const ImgDev* img_dev,
                       ImgCnt* cnt, int step, const DecEntry* lut)
{
    const int lat_w = (img_host->w + 1) / 2;
    const int lat_h = (img_host->h + 1) / 2;
    if (lat_h > 65535) return hipErrorInvalidValue;
    dim3 grid((lat_w + kThreads - 1) / kThreads, lat_h);
    if (img_host->dtype == 1)
        hipLaunchKernelGGL(k_step<uint8_t>, grid, dim3(kThreads), 0, stream, img_dev, cnt, step, lut);
    else
        hipLaunchKernelGGL(k_step<uint16_t>, grid, dim3(kThreads), 0, stream, img_dev, cnt, step, lut);
    return hipGetLastError();
}

// Compiled tile shapes: (tile height, tile width, halo = steps per residency,
// threads per tile, residency variant).
#define THIN_SHAPES(X)      \
    X(16, 16, 8, 256, 0)    \
    X(32, 32, 8, 256, 0)    \
    X(32, 32, 8, 512, 0)    \
    X(32, 32, 16, 256, 0)   \
    X(32, 32, 16, 1024, 0)  \
    X(32, 32, 16, 1024, 1)  \
    X(64, 64, 16, 1024, 0)  \
    X(64, 64, 16, 1024, 1)  \
    X(64, 64, 32, 1024, 0)  \
    X(64, 64, 8, 1024, 0)   \
    X(64, 64, 16, 512, 0)   \
    X(64, 64, 16, 256, 0)   \
    X(64, 64, 32, 512, 0)   \
    X(64, 64, 8, 512, 0)    \
    X(48, 48, 16, 512, 0)   \
    X(32, 32, 16, 512, 0)   \
    X(128, 128, 16, 512, 0) \
    X(128, 128, 16, 512, 1) \
    X(64, 64, 16, 512, 1)   \
    X(32, 32, 16, 256, 3)   \
    X(64, 64, 16, 256, 3)   \
    X(64, 64, 16, 256, 4)   \
    X(128, 128, 16, 256, 4) \
    X(32, 32, 16, 512, 3)   \
    X(64, 64, 16, 512, 3)   \
    X(64, 64, 16, 512, 4)   \
    X(64, 64, 32, 512, 3)   \
    X(64, 64, 32, 512, 4)   \
    X(128, 128, 16, 512, 3) \
    X(128, 128, 16, 512, 4) \
    X(128, 128, 32, 512, 4) \
    X(128, 128, 8, 512, 4)  \
    X(128, 128, 24, 512, 4) \
    X(64, 64, 16, 512, 2)   \
    X(32, 32, 16, 512, 2)   \
    X(16, 16, 8, 256, 2)    \
    X(16, 16, 16, 576, 2)   \
    X(16, 16, 16, 256, 2)   \
    X(24, 24, 12, 576, 2)   \
    X(16, 16, 16, 576, 0)   \
    X(32, 32, 8, 256, 2)    \
    X(32, 32, 16, 256, 2)   \
    X(32, 32, 16, 1024, 2)  \
    X(32, 32, 16, 1024, 5)  \
    X(32, 32, 16, 512, 5)   \
    X(32, 32, 32, 1024, 2)  \
    X(64, 64, 16, 1024, 2)  \
    X(64, 64, 32, 1024, 2)

bool tile_shape_supported(TileShape s)
{
#define X(a, b, c, n, e) \
    if (s.th == a && s.tw == b && s.k == c && s.nt == n && s.var == e) return true;
    THIN_SHAPES(X)
#undef X
    return false;
}

int compiled_shapes(TileShape* out, int cap)
{
    int n = 0;
#define X(a, b, c, t, e)                                  \
    if (n < cap && out) out[n] = TileShape{a, b, c, t, e}; \
    ++n;
    THIN_SHAPES(X)
#undef X
    return n;
}

TileShape complete_shape(int th, int tw, int k)
{
#define X(a, b, c, n, e) \
    if (th == a && tw == b && k == c) return TileShape{a, b, c, n, e};
    THIN_SHAPES(X)
#undef X
    return TileShape{0, 0, 0, 0, 0};
}

static int lds_bytes(TileShape s)
{
    if (s.var == kVarRegs || s.var == kVarRegsSeeded)
        return (s.th + 2 * s.k + 2) * (s.tw + 2 * s.k + 2) * 2 + 2048 + 64 +
               (s.var == kVarRegs ? 8 : 4 * (s.th + (s.th + 2 * s.k) * ((s.tw + 2 * s.k + 31) / 32 + 1)));
    const int region = (s.th + 2 * s.k) * (s.tw + 2 * s.k);
    const int hist = var_seeded(s.var)
                         ? (s.th * (s.tw / 32) + (s.th + 2 * s.k) * ((s.tw + 2 * s.k + 31) / 32)) * 4
                         : 8;
    if (s.var == kVarBits || s.var == kVarBitsSeeded) {
        const int lat_h = (s.th + 2 * s.k) / 2, lat_w = (s.tw + 2 * s.k) / 2;
        return region * 2 + 16 * lat_h * ((lat_w + 31) / 32) + 2 * lat_h * lat_w + 128 + 2048 + 64;
    }
    return region * 3 + hist + 2048 + 64;
}

int history_words(TileShape s) { return var_seeded(s.var) ? s.th * (s.tw / 32) : 1; }

int round_blocks_per_cu(TileShape s)
{
    const int by_lds = (160 * 1024) / lds_bytes(s);
    const int by_threads = 2048 / max(64, s.nt);
    return max(1, min(by_lds, by_threads));
}

hipError_t launch_round(hipStream_t stream, TileShape shape, const ImgDev* imgs, ImgCnt* cnt,
                        const int32_t* tile_img, int32_t* tile_last, int ntiles, int round,
                        const DecEntry* lut, int num_cus, uint32_t* hist_bits,
                        int32_t* hist_round, WorkList wl, const int32_t* round_base, int kflags)
{
    // The bit-flag variants keep u8 images as u8 in LDS: a launch with
    // kOnlyU8 takes that instantiation.
    const bool u8 = (kflags & kOnlyU8) != 0;
#define X(a, b, c, n, e)                                                                      \
    if (shape.th == a && shape.tw == b && shape.k == c && shape.nt == n && shape.var == e) {  \
        if constexpr (e == kVarBits || e == kVarBitsSeeded)                                   \
            if (u8)                                                                           \
                return launch_round_t<a, b, c, n, e, uint8_t>(stream, imgs, cnt, tile_img,    \
                                                              tile_last, ntiles, round, lut,   \
                                                              num_cus, hist_bits,              \
                                                              hist_round, wl, round_base,      \
                                                              kflags);                         \
        return launch_round_t<a, b, c, n, e, uint16_t>(stream, imgs, cnt, tile_img, tile_last, \
                                                       ntiles, round, lut, num_cus,             \
                                                       hist_bits, hist_round, wl, round_base,   \
                                                       kflags);                                 \
    }
    THIN_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_coop(hipStream_t stream, TileShape shape, const ImgDev* imgs, ImgCnt* cnt,
                       const int32_t* tile_img, int32_t* tile_last, int ntiles,
                       const DecEntry* lut, int32_t* active, int32_t* rounds_out,
                       int max_rounds, int num_cus, uint32_t* hist_bits, int32_t* hist_round,
                       int kflags)
{
    const bool u8 = (kflags & kOnlyU8) != 0;
#define X(a, b, c, n, e)                                                                      \
    if (shape.th == a && shape.tw == b && shape.k == c && shape.nt == n && shape.var == e) {  \
        if constexpr (e == kVarBits || e == kVarBitsSeeded)                                   \
            if (u8)                                                                           \
                return launch_coop_t<a, b, c, n, e, uint8_t>(stream, imgs, cnt, tile_img,     \
                                                             tile_last, ntiles, lut, active,   \
                                                             rounds_out, max_rounds, num_cus,  \
                                                             hist_bits, hist_round, kflags);   \
        return launch_coop_t<a, b, c, n, e, uint16_t>(stream, imgs, cnt, tile_img, tile_last,  \
                                                      ntiles, lut, active, rounds_out,          \
                                                      max_rounds, num_cus, hist_bits,           \
                                                      hist_round, kflags);                      \
    }
    THIN_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace thin
