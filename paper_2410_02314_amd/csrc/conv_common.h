// Pieces the residual network's convolution kernels share (kernels_conv.hip,
// kernels_split.hip): buffer resources, the decoded tile and its hand-over
// between waves.
#pragma once
#include "dloc_internal.h"

namespace dloc {

constexpr int NXCD = 8;
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

// Buffer resource over nbytes at base (raw addressing: stride 0, offsets in
// bytes).  A store whose offset lies past nbytes is dropped by the hardware,
// which lets the epilogue store without a branch around pixels off the frame;
// such a load reads zero.
constexpr uint32_t BUF_DWORD3 = 0x00020000u;
constexpr int BUF_OOB = (int)0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(void *base, uint32_t nbytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)nbytes, (int)BUF_DWORD3);
}

constexpr int align16(int b) { return (b + 15) / 16 * 16; }

__device__ __forceinline__ v4f relu4(v4f v)
{
    v4f r;
    r[0] = fmaxf(v[0], 0.f); r[1] = fmaxf(v[1], 0.f);
    r[2] = fmaxf(v[2], 0.f); r[3] = fmaxf(v[3], 0.f);
    return r;
}

// largest v (>= 0) of the four lanes j, j + 16, j + 32, j + 48, in each of them
// (register swaps between lane rows, where ds_bpermute would go through LDS)
__device__ __forceinline__ float lane_groups_max(float v)
{
    const int x = __float_as_int(v);
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const int y = max((int)a[0], (int)a[1]);       // non-negative floats order as integers
    const auto b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    return __int_as_float(max((int)b[0], (int)b[1]));
}

// ... and the sum, in the order (own + the lane group beside it) + the other two
__device__ __forceinline__ float lane_groups_sum(float v)
{
    const int x = __float_as_int(v);
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const int y = __float_as_int(__int_as_float((int)a[0]) + __int_as_float((int)a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    return __int_as_float((int)b[0]) + __int_as_float((int)b[1]);
}

// The fused 1x1 head (NH outputs of C channels, weights sH [NH][C]) over a wave's
// N pixel blocks, channel block by channel block: channels oc .. oc + 3 of the
// blocks' pixels into their sums.  The weights are read from LDS once for all N
// blocks (once per block, and with the lane sums through ds_bpermute, the head's
// layer of net B took, 4 x 2048^2: FP8 1008 us, now 926; BF16 1213, now 1184;
// FP32 2640, now 2574).
// head_blocks: how many of N blocks at a time keep the sums in registers (ten
// outputs, or 64 channels' accumulators, leave room for one).
template <int NH, int C> constexpr int head_blocks(int N) { return (NH > 5 || C > 48) && C > 16 ? 1 : N; }
template <int NH, int C, int N>
__device__ __forceinline__ void head_add(float (&hh)[N][NH], const float *sH, int oc, const v4f (&v)[N])
{
    v4f w[NH];
#pragma unroll
    for (int q = 0; q < NH; ++q) w[q] = *reinterpret_cast<const v4f *>(sH + q * C + oc);
#pragma unroll
    for (int p = 0; p < N; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int q = 0; q < NH; ++q) hh[p][q] += w[q][r] * v[p][r];
}
// The four lane groups hold disjoint channels of the pixel; group kq writes
// planes kq, kq + 4, kq + 8 (mp: the pixel in plane 0).
template <int NH>
__device__ __forceinline__ void head_store(float (&h)[NH], const float *bias, float *mp, int64_t plane, int kq, bool ok)
{
#pragma unroll
    for (int q = 0; q < NH; ++q) h[q] = lane_groups_sum(h[q]);
    if (ok) {
#pragma unroll
        for (int q = 0; q < NH; ++q)
            if ((q & 3) == kq) mp[q * plane] = h[q] + bias[q];
    }
}

// a decoded tile: origin (y0, x0) and size of its frame, where its input
// sits (point (ii, jj) of the tile is activation point a0 + ii rs + jj cs of
// the frame), and the frame's map and activation offsets
struct TileDec {
    int y0, x0, h, w, a0, rs, cs;
    int64_t px, act;
};

// Byte offsets of a tile's input (stride bytes a point) from its frame's first
// activation point, modulo 2^32: the tile's first halo point, and from there
// halo point (row, col).  A frame's points lie within 2^31 bytes of each other,
// so the sum is exact for every point of the frame, although the first halo point
// may lie up to 64 rows outside it (dilated plain rows) and the parts may wrap.
__host__ __device__ inline uint32_t halo_start(int a0, int rs, int cs, uint32_t stride)
{
    return ((uint32_t)a0 - (uint32_t)rs - (uint32_t)cs) * stride;
}
__host__ __device__ inline uint32_t halo_point(int row, int col, int rs, int cs, uint32_t stride)
{
    return ((uint32_t)row * (uint32_t)rs + (uint32_t)col * (uint32_t)cs) * stride;
}

// tile ti of the layer (of its active list in gated runs), in tr x tc tiles
__device__ __forceinline__ TileDec decode_conv_tile(const ConvArgs &a, const Geometry &geo, int nfr, int tr, int tc,
                                                    int64_t ti)
{
    const int dd = a.d, blk = a.blk;
    TileDec r;
    const int64_t t = a.list ? (int64_t)ld_const(a.list + ti) : ti;
    const int f = find_frame(a.fd, nfr, t, [blk](const FrameDesc &d) { return ld_const(&d.tile_start[blk]); });
    const FrameDesc *fd = a.fd + f;      // fields read in place: tile_start is indexed by the block
    r.h = ld_const(&fd->h);
    r.w = ld_const(&fd->w);
    r.px = ld_const(&fd->px_off);
    r.act = ld_const(&fd->act_off);
    decode_tile(r.h, r.w, t - ld_const(&fd->tile_start[blk]), dd, tr, tc, blk == geo.minor_blk, geo.strip, r.y0, r.x0);
    if (a.in_phase) {
        const int hd = (r.h + dd - 1) / dd, wd = (r.w + dd - 1) / dd;
        const int py = r.y0 % dd, px = r.x0 % dd;
        r.a0 = ((py * dd + px) * hd + r.y0 / dd) * wd + r.x0 / dd;
        r.rs = wd;
        r.cs = 1;
    } else {
        r.a0 = r.y0 * r.w + r.x0;
        r.rs = dd * r.w;
        r.cs = dd;
    }
    return r;
}

// Gated FP32 runs (pair kernels): did the layer before compute point (y, x) of the
// tile's frame?  An active tile also covers points that no layer computed in
// this run; what lies there is an earlier call's.  Nothing that is kept is made
// from them, but they would enter the largest magnitude, whose power of two all
// values of the tile share, so they read as zero.  (Frames are whole gate tiles,
// in order: the pixels before a frame give its first flag.)
__device__ __forceinline__ bool computed(const ConvArgs &a, const TileDec &t, int y, int x)
{
    const uint8_t *k = a.keep + t.px / (GATE_TILE * GATE_TILE);
    const int r = a.in_radius;
    if (2 * r >= GATE_TILE) return near_kept(k, t.h, t.w, y, y, x, x, r);
    // at most two gate tiles a side: all four flags at once, no loop (net B, 2 x
    // 2048^2 with 58 of 128 tiles kept: 10.47 ms -> 9.96; 9.69 without the test)
    const int g = t.w / GATE_TILE, ty0 = max(0, y - r) / GATE_TILE * g, ty1 = min(t.h - 1, y + r) / GATE_TILE * g;
    const int tx0 = max(0, x - r) / GATE_TILE, tx1 = min(t.w - 1, x + r) / GATE_TILE;
    return (k[ty0 + tx0] | k[ty0 + tx1] | k[ty1 + tx0] | k[ty1 + tx1]) != 0;
}

// Hand-over of a decoded tile through 64 bytes of LDS: one wave publishes it,
// every wave picks it up after the next barrier (into scalar registers).
__device__ __forceinline__ void publish_tile(int *slot, int lane, const TileDec &r)
{
    if (lane == 0) {
        int4 *q = reinterpret_cast<int4 *>(slot);
        q[0] = int4{r.y0, r.x0, r.h, r.w};
        q[1] = int4{r.a0, r.rs, r.cs, 0};
        q[2] = int4{(int)(uint32_t)r.px, (int)(r.px >> 32), (int)(uint32_t)r.act, (int)(r.act >> 32)};
    }
}

__device__ __forceinline__ TileDec pickup_tile(const int *slot)
{
    const int4 *q = reinterpret_cast<const int4 *>(slot);
    const int4 u0 = q[0], u1 = q[1], u2 = q[2];
    TileDec r;
    r.y0 = __builtin_amdgcn_readfirstlane(u0.x);
    r.x0 = __builtin_amdgcn_readfirstlane(u0.y);
    r.h = __builtin_amdgcn_readfirstlane(u0.z);
    r.w = __builtin_amdgcn_readfirstlane(u0.w);
    r.a0 = __builtin_amdgcn_readfirstlane(u1.x);
    r.rs = __builtin_amdgcn_readfirstlane(u1.y);
    r.cs = __builtin_amdgcn_readfirstlane(u1.z);
    r.px = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane(u2.x) |
           ((int64_t)__builtin_amdgcn_readfirstlane(u2.y) << 32);
    r.act = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane(u2.z) |
            ((int64_t)__builtin_amdgcn_readfirstlane(u2.w) << 32);
    return r;
}

// Division of 32-bit values by a divisor that changes rarely: with m =
// floor((2^32 - 1) / d), the high word of n m is floor(n / d) or one less
struct UDiv {
    uint32_t d, m;
    __device__ __forceinline__ void set(uint32_t div) { d = div; m = 0xFFFFFFFFu / div; }
    __device__ __forceinline__ uint32_t div(uint32_t n) const
    {
        const uint32_t q = __umulhi(n, m);
        return n - q * d >= d ? q + 1 : q;
    }
};

// Decoder of a layer's conv tiles (tr x tc) that keeps what depends on the
// frame alone -- its tile range, sizes and the divisors of decode_tile -- and
// so takes a few scalar instructions per tile while consecutive tiles stay in
// one frame.  Every wave runs its own: a layer of one wave per SIMD has no
// other wave to hide one wave's decoding behind.
struct TileWalk {
    int64_t ts0 = 1, ts1 = 0;           // the frame's tiles (empty: no frame yet)
    int64_t px, act;
    int h, w, hd, wd;                   // frame, and its phase sub-images
    uint32_t rxn, strip;
    UDiv a, b, c, last, dd;             // phase-major: regions, strip tiles, strip and last strip width; minor: d^2, rxn

    template <class Args> __device__ __forceinline__ void frame(const Args &ca, const Geometry &geo, int nfr, int tr, int tc, int64_t t)
    {
        const int blk = ca.blk, d = ca.d;
        const int f = find_frame(ca.fd, nfr, t, [blk](const FrameDesc &x) { return ld_const(&x.tile_start[blk]); });
        const FrameDesc *fd = ca.fd + f;
        ts0 = ld_const(&fd->tile_start[blk]);
        ts1 = f + 1 < nfr ? ld_const(&fd[1].tile_start[blk]) : INT64_MAX;
        h = ld_const(&fd->h);
        w = ld_const(&fd->w);
        px = ld_const(&fd->px_off);
        act = ld_const(&fd->act_off);
        hd = (h + d - 1) / d;
        wd = (w + d - 1) / d;
        const uint32_t ryn = (uint32_t)((h + tr * d - 1) / (tr * d));
        rxn = (uint32_t)((w + tc * d - 1) / (tc * d));
        strip = geo.strip;
        dd.set((uint32_t)d);
        if (blk == geo.minor_blk) {
            a.set((uint32_t)(d * d));
            b.set(rxn);
            c = last = b;
        } else {
            a.set(ryn * rxn);
            b.set(ryn * strip);
            c.set(strip);
            last.set(rxn - (rxn - 1) / strip * strip);
        }
    }
    template <class Args> __device__ __forceinline__ TileDec tile(const Args &ca, const Geometry &geo, int nfr, int tr, int tc, int64_t ti)
    {
        const int64_t t = ca.list ? (int64_t)ld_const(ca.list + ti) : ti;
        if (t < ts0 || t >= ts1) frame(ca, geo, nfr, tr, tc, t);
        const uint32_t l = (uint32_t)(t - ts0), d = (uint32_t)ca.d;
        uint32_t ph, ry, rx;
        if (ca.blk == geo.minor_blk) {
            const uint32_t r = a.div(l);
            ph = l - r * a.d;
            ry = b.div(r);
            rx = r - ry * rxn;
        } else {
            ph = a.div(l);
            const uint32_t r = l - ph * a.d;
            const uint32_t st = b.div(r), in = r - st * b.d;
            const bool tail = (st + 1) * strip >= rxn;
            UDiv sw;
            sw.d = tail ? last.d : c.d;
            sw.m = tail ? last.m : c.m;
            ry = sw.div(in);
            rx = st * strip + (in - ry * sw.d);
        }
        const uint32_t py = dd.div(ph), pxl = ph - py * d;
        TileDec r;
        r.y0 = (int)(ry * (uint32_t)tr * d + py);
        r.x0 = (int)(rx * (uint32_t)tc * d + pxl);
        r.h = h;
        r.w = w;
        r.px = px;
        r.act = act;
        // (a tile's first row and column of its phase's sub-image: ry tr, rx tc)
        r.a0 = ca.in_phase ? ((int)ph * hd + (int)ry * tr) * wd + (int)rx * tc : r.y0 * w + r.x0;
        r.rs = ca.in_phase ? wd : (int)d * w;
        r.cs = ca.in_phase ? 1 : (int)d;
        return r;
    }
};

// ---- the FP32 form's layers of up to 48 channels (kernels_split.hip): activations in planes of 16 channels ----
bool split_takes(int C, int precision);
size_t split_packed_bytes(int C);       // a layer's fragments (split_pack_group: channels of a K group), then its FP32 weights
inline int split_pack_group(int C) { return C == 32 ? 32 : 16; }
int split_max_grid(int C, int tr, int ncu);
hipError_t launch_split(int C, const ConvArgs &a, const Geometry &g, int grid, hipStream_t s);

// ---- a residual block's two BF16 layers in one kernel (kernels_block.hip) ----
struct BlockArgs {
    ConvArgs c;              // the second layer's; in: the block's input, which is also the residual
    const void *w1;          // the first layer's packed weights and bias
    const float *b1;
};
bool block_takes(int C, int precision, int tr, int64_t tiles, int ncu);
hipError_t launch_block(int C, const BlockArgs &a, const Geometry &g, int ncu, hipStream_t s);

}  // namespace dloc
