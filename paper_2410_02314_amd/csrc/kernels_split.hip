// 3x3 dilated convolution layers of the FP32 form (to 48 channels) on the
// FP16 matrix cores (gfx950).
//
// Operation: as kernels_conv.hip (paper Sec. 3.2.1, dilated convolution; Sec.
// 3.2, per-pixel head): y[p][o] = b[o] + sum_{tap, c} W[o][c][tap] *
// x[p + d off(tap)][c], optional residual, ReLU, optional fused 1x1 head.
//
// Products.  Every FP32 operand is held as two FP16 halves, hi = f16(v 2^s) and
// lo = f16((v 2^s - hi) 2^11): 22 significant bits and the sign of lo.  A
// product is taken as wh xh + (wh xl + wl xh) 2^-11, the two sums in FP32
// accumulators of their own.  The operand error (2^-23 of the value at most)
// lies below the rounding of an FP32 accumulation over 9 C products, and here
// a sum is rounded once per 32 products instead of once per product: on whole
// nets the error against 64-bit arithmetic is 2.3e-7 of the maps' norm (48
// channels, 10 layers), and was 3.9e-7 with v_mfma_f32_16x16x4_f32; over 31 random
// residual and dense nets it is 0.72 times that form's (0.95 at most).
// Three FP16 MFMAs take 3/16 of the cycles of the FP32 MFMAs they replace.
//   Range: s brings the largest input of a tile into [2^14, 2^15) (exact powers of
// two); values down to 2^-28 of it keep all 22 bits, smaller ones are off by 2^-50
// of it at most.  (While s moved in steps of 20, a tile with one value past 2^15
// kept 2^-16 absolute: 9.5e-6 of the sums beside it, where FP32 products added one
// by one give 3.1e-7 and these steps 7.5e-8.)  A magnitude below 2^-46 as the
// tile's largest leaves fewer bits (s is 60 at most): 2^-31 of it at 2^-65.  Weights
// are scaled in the same way by a power of two per output channel.  A tile holding
// an infinity or a value of 2^75 or more, or nothing but values below 2^-65 (or any
// tile of a layer whose weights are of such magnitudes) takes plain FP32 FMAs
// instead (slow_tile), so those come out as in FP32; NaNs propagate by themselves.
//
// Tiling.  Tiles, persistent workgroups and XCD ranges as in kernels_conv.hip:
// TR x 32 output points per tile.  A wave computes 16 columns of R rows for all
// output channels.  One K step takes 32 values of one tap row u: an input row's
// fragment is read from LDS once per step and multiplied into the (up to three)
// output rows it belongs to, and a weight fragment once for the wave's R rows.
//
// Activations in HBM and LDS lie in planes of 16 channels, 64 bytes per point
// and plane in HBM: a wave stores 16 points x 16 channels as 1 KB of whole
// lines, and a group's tile rows are contiguous.  (In NHWC with 48 channels
// those stores are 64-byte pieces 192 bytes apart: 2.33 ms against 2.18.)  In
// LDS a plane holds 32 bytes per point, hi or lo: a point stride of 8 dwords,
// which a 16-byte read of 16 points x 2 channel halves serves without bank
// conflicts, and no padding.
//
// Two kernels:
//   k_split (16 and 32 channels) stages a tile's hi and lo planes at once, four
// waves of R = TR / 2 rows; weights and tile take 80 KB (32 channels, 8 rows),
// so two workgroups share a CU and hide each other's conversion and epilogue.
//   k_pipe (48 channels) has 86 KB of weights and room for one workgroup, so it
// walks K in groups of 16 channels through two LDS buffers: while the MFMAs of
// one group run, the next group is converted into the other buffer and the
// loads three groups on are in flight, with one barrier per group.  TR waves of
// R = 2 rows, two per SIMD.  The tile's exponent is then known group by group:
// a later group that needs a lower one has the sums so far rescaled.
//
// Measured (mean launch without head, 4 x 2048^2 points): 48 channels 5.11 ms
// with FP32 MFMAs, 2.32 ms as k_split, 2.18 ms as k_pipe; 32 channels 2.40 and
// 1.15 ms.  Bounds: the HBM bytes take 1.5 and 1.0 ms at the 5.2 TB/s of a copy;
// the MFMAs of 48 channels 1.4 ms at the 1.66 PFLOP/s that chains of this MFMA
// sustain with two waves per SIMD (24 cycles each, not 16), and the clock falls
// from 2.4 to 1.9 GHz under them.
#include <algorithm>
#include <type_traits>

#include "conv_common.h"
#include "split_common.h"

namespace dloc {

namespace {

constexpr int TC = 32, PW = TC + 2, NTH = 256;

// A tile of 4 rows takes the power of two of the tile of 8 rows it is half of, so
// that a frame gives the same bits with either (the rows depend on the batch, the
// config and the autotuner): it also reads the other half's rows, four more of
// each group, for their largest magnitude alone (4 x 128^2, net A: 2.4 us of a
// graph replay's 93).  extra_point: point e of these
// as row and column of its own halo (row 0: the first halo row).
constexpr int NEXTRA = 4 * PW;
__device__ __forceinline__ void extra_point(int e, bool odd, int &row, int &col)
{
    const int r = e / PW;
    col = e - r * PW;
    row = r + (odd ? -4 : 6);
}

// K plan: per tap row u, 3 taps x C channels in chunks of 8 (tap column major),
// taken four at a time; with 2 chunks left over (16 channels) two closing
// steps share them among the tap rows: step 0 holds those of u = 0 (lane
// groups 0, 1) and u = 1 (2, 3), step 1 those of u = 2 and zero weights
template <int C> struct SPlan {
    static constexpr int CH8 = C / 8, NB = C / 16;
    static constexpr int FULL = 3 * CH8 / 4;
    static constexpr bool HALF = 3 * CH8 % 4 != 0;
    static constexpr int NSTEP = 3 * FULL + (HALF ? 2 : 0);      // weight steps
    static constexpr int WBYTES = NSTEP * NB * 2 * 64 * 16;      // hi and lo fragments
};

template <int C, int TR, int NH> struct SLds {
    static constexpr int NPT = (TR + 2) * PW;
    static constexpr int PLANE = NPT * 32;                       // 16 channels of every point
    static constexpr int LO = PLANE * (C / 16);                  // lo planes after the hi planes
    static constexpr int WOFF = 2 * LO;
    static constexpr int BOFF = WOFF + SPlan<C>::WBYTES;         // bias [C]
    static constexpr int SOFF = BOFF + C * 4;                    // weight scales [C]
    static constexpr int HOFF = SOFF + C * 4;                    // head [NH C + NH]
    static constexpr int MOFF = align16(HOFF + (NH * C + NH) * 4);   // wave maxima [4]
    static constexpr int TOTAL = MOFF + 16;
    static constexpr bool FITS = TOTAL <= 160 * 1024;
};

// One tile in plain FP32 FMAs, a thread per output point, in tap and channel
// order, from HBM and the unpacked weights: the rare tile whose values the FP16
// halves cannot hold (an infinity, or a magnitude past their scaling).
template <int C, int TR, int NH>
__device__ __forceinline__ void slow_tile(const ConvArgs &a, const TileDec &n, const float *gw, const float *sB,
                                          const float *sH)
{
    const int dd = a.d, row = threadIdx.x / TC, col = threadIdx.x % TC;
    const int yo = n.y0 + dd * row, xo = n.x0 + dd * col;
    if (row >= TR || yo >= n.h || xo >= n.w) return;
    const char *gx = static_cast<const char *>(a.in) + n.act * a.pstride;
    const int64_t ipt = n.a0 + (int64_t)row * n.rs + col * n.cs;
    const int osh = a.out_shift, om = (1 << osh) - 1;
    const int64_t opt = n.act + ((((yo & om) << osh) + (xo & om)) * (int64_t)((n.h + om) >> osh) + (yo >> osh)) *
                                    ((n.w + om) >> osh) + (xo >> osh);
    float hh[NH > 0 ? NH : 1] = {};
#pragma unroll 1
    for (int oc = 0; oc < C; ++oc) {
        float s = 0.f;
#pragma unroll 1
        for (int tap = 0; tap < 9; ++tap) {
            const int u = tap / 3 - 1, v = tap % 3 - 1, yy = yo + dd * u, xx = xo + dd * v;
            if ((unsigned)yy >= (unsigned)n.h || (unsigned)xx >= (unsigned)n.w) continue;
            const char *xp = gx + (ipt + u * n.rs + v * n.cs) * a.pstride;
#pragma unroll 1
            for (int c = 0; c < C; ++c)
                s = fmaf(gw[(oc * C + c) * 9 + tap], *reinterpret_cast<const float *>(xp + (c >> 4) * a.gstride + (c & 15) * 4), s);
        }
        s += sB[oc];
        const int64_t co = (oc >> 4) * a.gstride + (oc & 15) * 4;
        if (a.res) s += *reinterpret_cast<const float *>(static_cast<const char *>(a.res) + (n.act + ipt) * a.pstride + co);
        s = fmaxf(s, 0.f);
        if constexpr (NH == 0) *reinterpret_cast<float *>(static_cast<char *>(a.out) + opt * a.pstride + co) = s;
#pragma unroll
        for (int q = 0; q < NH; ++q) hh[q] += sH[q * C + oc] * s;
    }
#pragma unroll
    for (int q = 0; q < NH; ++q)
        a.maps[NH * n.px + ((int64_t)q * n.h + yo) * n.w + xo] = hh[q] + sH[NH * C + q];
}

template <int C, int TR, bool RES, int NH, bool GATED>
__global__ void __launch_bounds__(NTH, 2)
k_split(ConvArgs a, Geometry geo)
{
    constexpr bool HEAD = NH > 0;
    using L = SLds<C, TR, (NH > 5 ? NH : 5)>;
    using K = SPlan<C>;
    constexpr int NB = K::NB, R = TR / 2, NPT = L::NPT;
    extern __shared__ v4f smem[];
    char *sT = reinterpret_cast<char *>(smem);
    float *sB = reinterpret_cast<float *>(sT + L::BOFF);
    float *sS = reinterpret_cast<float *>(sT + L::SOFF);
    float *sH = reinterpret_cast<float *>(sT + L::HOFF);
    float *sM = reinterpret_cast<float *>(sT + L::MOFF);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: keeps row state scalar
    const int j = lane & 15, kq = lane >> 4, kh = kq >> 1;
    const int strip = wave & 1, row0 = (wave >> 1) * R;
    const int dd = a.d, blk = a.blk;

    {
        const v4f *gw = static_cast<const v4f *>(a.wpk);
        v4f *sW = reinterpret_cast<v4f *>(sT + L::WOFF);
#pragma unroll 6
        for (int i = tid; i < K::WBYTES / 16; i += NTH) sW[i] = gw[i];
    }
    for (int i = tid; i < C; i += NTH) {
        sB[i] = a.bias[i];
        sS[i] = a.wscale[i];
    }
    // a layer whose weights the FP16 halves cannot hold has scale 0
    const bool slow_layer = ld_const(a.wscale) == 0.f;
    if (HEAD)
        for (int i = tid; i < NH * C + NH; i += NTH) sH[i] = a.head[i];

    const int64_t T = a.list ? (int64_t)ld_const(a.list_count)
                      : geo.dyn ? ld_const(geo.dyn + DYN_TILES + blk) : geo.tiles[blk];
    const int nfr = geo.dyn ? (int)ld_const(geo.dyn + DYN_NF) : geo.nf;
    const int xcd = blockIdx.x % NXCD, slot = blockIdx.x / NXCD, nslot = gridDim.x / NXCD;
    const int64_t chunk = (T + NXCD - 1) / NXCD;
    const int64_t t0 = (int64_t)xcd * chunk;
    const int64_t t1 = t0 + chunk < T ? t0 + chunk : T;

    // the next tile's input in registers (off-frame points take an
    // out-of-range buffer offset and read zero)
    constexpr int NQ = NPT * 4;              // 16-byte chunks of 16 channels of the tile's points
    constexpr int NPF = (NQ + NTH - 1) / NTH;
    v4f pf[NB][NPF];
    constexpr int NPE = TR == 4 ? (NEXTRA * 4 + NTH - 1) / NTH : 0;
    v4f pe[NB][NPE > 0 ? NPE : 1];           // [TR 4] the other half's rows
    TileWalk walk;
    auto decode = [&](int64_t ti) { return walk.tile(a, geo, nfr, TR, TC, ti); };
    // byte offsets of this thread's chunks from the tile's first halo point:
    // they depend on the frame's row stride alone
    int off[NPF], off_rs = -1;
    auto issue = [&](const TileDec &r) {
        if (r.rs != off_rs) {
            off_rs = r.rs;
            int tv = tid;
            asm volatile("" : "+v"(tv));     // (worked out here, its parts not kept over the whole loop)
#pragma unroll
            for (int k = 0; k < NPF; ++k) {
                const int q = tv + k * NTH, pt = q >> 2;
                off[k] = (int)halo_point(pt / PW, pt - pt / PW * PW, r.rs, r.cs, (uint32_t)a.pstride) + (q & 3) * 16;
            }
        }
        // from the frame's first point, or, an interior tile's points all lying in
        // the frame, from the first of them
        char *const frame = const_cast<char *>(static_cast<const char *>(a.in)) + r.act * a.pstride;
        char *p = frame;
        const uint32_t start = halo_start(r.a0, r.rs, r.cs, (uint32_t)a.pstride);
        const bool inside = !GATED && r.y0 >= dd && r.y0 + dd * TR < r.h && r.x0 >= dd && r.x0 + dd * TC < r.w;
        int o[NPF];
        if (inside) {
            p += start;
#pragma unroll
            for (int k = 0; k < NPF; ++k) o[k] = (k + 1) * NTH <= NQ || tid + k * NTH < NQ ? off[k] : BUF_OOB;
        } else {
            int tv = tid;
            asm volatile("" : "+v"(tv));     // (worked out here, not kept in registers over the whole loop)
#pragma unroll
            for (int k = 0; k < NPF; ++k) {
                const int q = tv + k * NTH, pt = q >> 2;
                const int y = r.y0 + dd * (pt / PW - 1), x = r.x0 + dd * (pt - pt / PW * PW - 1);
                const bool ok = (q < NQ) & ((unsigned)y < (unsigned)r.h) & ((unsigned)x < (unsigned)r.w);
                o[k] = ok && (!GATED || computed(a, r, y, x)) ? (int)((uint32_t)off[k] + start) : BUF_OOB;
            }
        }
#pragma unroll
        for (int g = 0; g < NB; ++g)
#pragma unroll
            for (int k = 0; k < NPF; ++k)
                pf[g][k] = __builtin_bit_cast(
                    v4f, __builtin_amdgcn_raw_buffer_load_b128(buf_rsrc(p + g * a.gstride, 0x7FFFFFFFu), o[k], 0, 0));
        if constexpr (NPE > 0) {
            const bool odd = walk.dd.div((uint32_t)r.y0) & 4u;
#pragma unroll
            for (int k = 0; k < NPE; ++k) {
                const int q = tid + k * NTH;
                int row, col;
                extra_point(q >> 2, odd, row, col);
                const int y = r.y0 + dd * (row - 1), x = r.x0 + dd * (col - 1);
                bool ok = (q < NEXTRA * 4) & ((unsigned)y < (unsigned)r.h) & ((unsigned)x < (unsigned)r.w);
                if constexpr (GATED) ok = ok && computed(a, r, y, x);
                const int oe = ok ? (int)(start + halo_point(row, col, r.rs, r.cs, (uint32_t)a.pstride)) + (q & 3) * 16 : BUF_OOB;
#pragma unroll
                for (int g = 0; g < NB; ++g)
                    pe[g][k] = __builtin_bit_cast(
                        v4f, __builtin_amdgcn_raw_buffer_load_b128(buf_rsrc(frame + g * a.gstride, 0x7FFFFFFFu), oe, 0, 0));
            }
        }
    };

    // n: the current tile; nx: the next one
    TileDec n{}, nx{};
    int64_t ti = t0 + slot;
    if (ti < t1) {
        nx = decode(ti);
        issue(nx);
    }
    // the first tile's data is waited for outside the loop, so that the wait at
    // the loop top covers the loop's own path only
#pragma unroll
    for (int g = 0; g < NB; ++g)
#pragma unroll
        for (int k = 0; k < NPF; ++k) asm volatile("" : : "v"(pf[g][k]));

    // LDS addresses: this lane's MFMA operand (point (row0, 16 strip + j) of the
    // tile, channel half kq & 1 of plane 0; its weight fragment) and this
    // thread's staging chunks
    const char *xb = sT + (row0 * PW + 16 * strip + j) * 32 + (kq & 1) * 16;
    const char *wb = sT + L::WOFF + lane * 16;
    char *stage = sT + (tid >> 2) * 32 + (tid & 3) * 8;
    // offset of chunk pair q (16 channels of one tap) of a tap row
    auto pair_off = [](int q) { return (2 * q / K::CH8) * 32 + (2 * q % K::CH8 / 2) * L::PLANE; };

    for (; ti < t1; ti += nslot) {
        n = nx;
        if (ti + nslot < t1) nx = decode(ti + nslot);
        const int Y0 = n.y0, X0 = n.x0, H = n.h, W = n.w;

        // the tile's largest magnitude sets its power of two
        float mx = 0.f;
#pragma unroll
        for (int g = 0; g < NB; ++g)
#pragma unroll
            for (int k = 0; k < NPF; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, fabsf(pf[g][k][r]));
#pragma unroll
        for (int g = 0; g < NB; ++g)
#pragma unroll
            for (int k = 0; k < NPE; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, fabsf(pe[g][k][r]));
        mx = wave_max(mx);
        if (lane == 0) sM[wave] = mx;
        __syncthreads();   // the previous tile's LDS reads are done (and weights staged, maxima written)
        const v4f mv = *reinterpret_cast<const v4f *>(sM);
        const uint32_t mb = (uint32_t)__builtin_amdgcn_readfirstlane(
            __float_as_int(fmaxf(fmaxf(mv[0], mv[1]), fmaxf(mv[2], mv[3]))));
        const bool slow = slow_layer | split_misfit(mb);
        const int sexp = split_exp(mb);
        const float sc = __int_as_float((127 + sexp) << 23);
#pragma unroll
        for (int i = 0; i < NB * NPF; ++i) {
            const int g = i % NB, k = i / NB;
            if ((k + 1) * NTH > NQ && tid + k * NTH >= NQ) continue;
            split_store(pf[g][k] * sc, L::LO, stage + g * L::PLANE + k * (NTH / 4 * 32));
        }
        __syncthreads();

        // the residual at this wave's output points (off-frame points read
        // zero), then the next tile's input: in order, so waiting for the
        // residual does not wait for the prefetch
        v4f rr[RES ? R : 1][RES ? NB : 1];
        const int xo = X0 + dd * (16 * strip + j);
        if constexpr (RES) {
            __amdgpu_buffer_rsrc_t rres[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                rres[nb] = buf_rsrc(const_cast<char *>(static_cast<const char *>(a.res)) + n.act * a.pstride + nb * a.gstride,
                                    0x7FFFFFFFu);
#pragma unroll
            for (int y = 0; y < R; ++y) {
                const bool ok = (Y0 + dd * (row0 + y) < H) & (xo < W);
                const int o = ok ? (n.a0 + (row0 + y) * n.rs + (16 * strip + j) * n.cs) * (int)a.pstride + kq * 16 : BUF_OOB;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    rr[y][nb] = __builtin_bit_cast(
                        v4f, __builtin_amdgcn_raw_buffer_load_b128(rres[nb], o, 0, 0));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // (past the last tile nothing is loaded: of a few tiles per workgroup such
        // loads are a good part; net A, 4 x 128^2 90.0 -> 87.7 us, 517 x 600 205.7 ->
        // 200.7, full frames as before)
        if (ti + nslot < t1) issue(nx);
        __builtin_amdgcn_sched_barrier(0);
        if (slow) {
            slow_tile<C, TR, NH>(a, n, reinterpret_cast<const float *>(static_cast<const char *>(a.wpk) + K::WBYTES), sB, sH);
            continue;
        }

        v4f acc[R][NB], acx[R][NB];                       // wh xh; the cross sums
#pragma unroll
        for (int y = 0; y < R; ++y)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[y][nb] = acx[y][nb] = v4f{0.f, 0.f, 0.f, 0.f};
        // operands, hi and lo: x the fragments of K step m, one per input row
        // (the closing steps: one per output row), w weight step s
        v4f x[R + 2][2], w[NB][2];
        auto load_x = [&](int m) {
            const bool closing = m >= K::FULL;           // rows y (u = 0) and y + 1 (u = 1); then row y + 2 (u = 2)
            const char *p = xb + (closing ? pair_off(2 * K::FULL) + (m == K::FULL ? kh * (PW * 32) : 2 * (PW * 32))
                                          : kh ? pair_off(2 * m + 1) : pair_off(2 * m));
#pragma unroll
            for (int y = 0; y < (closing ? R : R + 2); ++y) {
                x[y][0] = *reinterpret_cast<const v4f *>(p + y * (PW * 32));
                x[y][1] = *reinterpret_cast<const v4f *>(p + y * (PW * 32) + L::LO);
            }
        };
        auto load_w = [&](int s) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int h = 0; h < 2; ++h) w[nb][h] = *reinterpret_cast<const v4f *>(wb + ((s * NB + nb) * 2 + h) * 1024);
        };
#pragma unroll
        for (int s = 0; s < K::NSTEP; ++s) {
            const int m = s < 3 * K::FULL ? s / 3 : s - 2 * K::FULL, u = s < 3 * K::FULL ? s % 3 : 0;
            if (m >= K::FULL || u == 0) load_x(m);
            load_w(s);
            __builtin_amdgcn_sched_barrier(0);       // issued before this step's MFMAs
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int y = 0; y < R; ++y)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const v4f wv = w[nb][t == 2], xv = x[y + u][t == 1];
                        v4f &d = t > 0 ? acx[y][nb] : acc[y][nb];
                        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, wv), __builtin_bit_cast(v8h, xv),
                                                                   d, 0, 0, 0);
                    }
            __builtin_amdgcn_sched_barrier(0);
        }

        // epilogue: D row = output channel 16 nb + 4 kq + r, column = pixel j.
        // Stores go through a buffer resource; pixels past the frame edge take
        // an out-of-range offset and are dropped.
        const int osh = a.out_shift, om = (1 << osh) - 1;
        const int ohd = (H + om) >> osh, owd = (W + om) >> osh;
        __amdgpu_buffer_rsrc_t orow[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            orow[nb] = buf_rsrc(HEAD ? nullptr : static_cast<char *>(a.out) + n.act * a.pstride + nb * a.gstride,
                                HEAD ? 0u : 0x7FFFFFFFu);
        const float ts = __int_as_float((127 - sexp) << 23);
        v4f bias[NB], scl[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            bias[nb] = *reinterpret_cast<const v4f *>(sB + nb * 16 + kq * 4);
            scl[nb] = *reinterpret_cast<const v4f *>(sS + nb * 16 + kq * 4) * ts;
        }
        auto value = [&](int y, int nb) {
            v4f v = acc[y][nb];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = fmaf(fmaf(acx[y][nb][r], 0x1p-11f, v[r]), scl[nb][r], bias[nb][r]);
                if constexpr (RES) v[r] += rr[y][nb][r];
            }
            return relu4(v);
        };
        if constexpr (HEAD) {
            constexpr int N = head_blocks<NH, C>(R);
#pragma unroll
            for (int y0 = 0; y0 < R; y0 += N) {
                float hh[N][NH] = {};                // head sums of this lane's channels
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    v4f vr[N];
#pragma unroll
                    for (int y = 0; y < N; ++y) vr[y] = value(y0 + y, nb);
                    head_add<NH, C>(hh, sH, nb * 16 + kq * 4, vr);
                }
#pragma unroll
                for (int y = 0; y < N; ++y) {
                    const int yo = Y0 + dd * (row0 + y0 + y);
                    head_store(hh[y], sH + NH * C, a.maps + NH * n.px + (int64_t)yo * W + xo, (int64_t)H * W, kq, (yo < H) & (xo < W));
                }
            }
        } else {
#pragma unroll
            for (int y = 0; y < R; ++y) {
                const int yo = Y0 + dd * (row0 + y);
                const bool ok = (yo < H) & (xo < W);
                const int opt = ((((yo & om) << osh) + (xo & om)) * ohd + (yo >> osh)) * owd + (xo >> osh);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, value(y, nb)), orow[nb],
                                                           ok ? opt * (int)a.pstride + kq * 16 : BUF_OOB, 0, 0);
            }
        }
    }
}

// ---- pipelined by channel group ----
// LDS: two buffers of one 16-channel group's tile (hi and lo planes), all
// weights, the per-channel constants, the wave maxima of two groups
template <int C, int TR, int NH> struct PLds {
    static constexpr int NPT = (TR + 2) * PW;
    // (room for the chunks of the threads past the last point)
    static constexpr int PLANE = (NPT + 16 * TR - 1) / (16 * TR) * (16 * TR) * 32, BUF = 2 * PLANE;
    static constexpr int WBYTES = C / 16 * 5 * (C / 16) * 2048;
    static constexpr int WOFF = 2 * BUF;
    static constexpr int BOFF = WOFF + WBYTES;
    static constexpr int SOFF = BOFF + C * 4;
    static constexpr int HOFF = SOFF + C * 4;
    static constexpr int MOFF = align16(HOFF + (NH * C + NH) * 4);   // wave maxima [2][8]
    static constexpr int TOTAL = MOFF + 64;
    static constexpr bool FITS = TOTAL <= 160 * 1024;
};

template <int C, int TR, bool RES, int NH, bool GATED>
__global__ void __launch_bounds__(TR * 64, 2)
k_pipe(ConvArgs a, Geometry geo)
{
    constexpr bool HEAD = NH > 0;
    using L = PLds<C, TR, (NH > 5 ? NH : 5)>;
    constexpr int R = 2, NTH = TR * 64, NB = C / 16, G = C / 16, NPT = L::NPT;
    extern __shared__ v4f smem[];
    char *sT = reinterpret_cast<char *>(smem);
    float *sB = reinterpret_cast<float *>(sT + L::BOFF);
    float *sS = reinterpret_cast<float *>(sT + L::SOFF);
    float *sH = reinterpret_cast<float *>(sT + L::HOFF);
    float *sM = reinterpret_cast<float *>(sT + L::MOFF);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kq = lane >> 4, kh = kq >> 1;
    const int strip = wave & 1, row0 = (wave >> 1) * R;
    const int dd = a.d, blk = a.blk;
    {
        const v4f *gw = static_cast<const v4f *>(a.wpk);
        v4f *sW = reinterpret_cast<v4f *>(sT + L::WOFF);
#pragma unroll 6
        for (int i = tid; i < L::WBYTES / 16; i += NTH) sW[i] = gw[i];
    }
    for (int i = tid; i < C; i += NTH) {
        sB[i] = a.bias[i];
        sS[i] = a.wscale[i];
    }
    const bool slow_layer = ld_const(a.wscale) == 0.f;
    if (HEAD)
        for (int i = tid; i < NH * C + NH; i += NTH) sH[i] = a.head[i];

    const int64_t T = a.list ? (int64_t)ld_const(a.list_count)
                      : geo.dyn ? ld_const(geo.dyn + DYN_TILES + blk) : geo.tiles[blk];
    const int nfr = geo.dyn ? (int)ld_const(geo.dyn + DYN_NF) : geo.nf;
    const int xcd = blockIdx.x % NXCD, slot = blockIdx.x / NXCD, nslot = gridDim.x / NXCD;
    const int64_t chunk = (T + NXCD - 1) / NXCD;
    const int64_t t0 = (int64_t)xcd * chunk;
    const int64_t t1 = t0 + chunk < T ? t0 + chunk : T;
    int64_t ti = t0 + slot;
    if (ti >= t1) return;

    // staging: chunk k of a thread is 4 channels (16 bytes) of one point of the
    // group's tile; rows and columns as multiples of d, offsets from the tile's
    // first halo point (which change with the frame's row stride)
    constexpr int NQ = NPT * 4, NPF = (NQ + NTH - 1) / NTH;
    v4f pf[3][NPF];
    constexpr int NPE = TR == 4 ? (NEXTRA * 4 + NTH - 1) / NTH : 0;
    v4f pe[NPE > 0 ? NPE : 1];             // [TR 4] the other half's rows of one group
    int off[NPF], dy[NPF], dx[NPF], off_rs = -1;
    char *stage = sT + (tid >> 2) * 32 + (tid & 3) * 8;
#pragma unroll
    for (int k = 0; k < NPF; ++k) {
        const int q = tid + k * NTH, pt = q >> 2;
        dy[k] = q < NQ ? dd * (pt / PW) : 1 << 30;       // past the last chunk: off every frame
        dx[k] = dd * (pt - pt / PW * PW);
    }
    TileWalk walk;
    auto decode = [&](int64_t t) { return walk.tile(a, geo, nfr, TR, TC, t < t1 ? t : t1 - 1); };
    auto offsets = [&](const TileDec &r) {
        if (r.rs == off_rs) return;
        off_rs = r.rs;
        int tv = tid;
        asm volatile("" : "+v"(tv));         // (as in k_split)
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const int q = tv + k * NTH, pt = q >> 2;
            off[k] = (int)halo_point(pt / PW, pt - pt / PW * PW, r.rs, r.cs, (uint32_t)a.pstride) + (q & 3) * 16;
        }
    };
    struct Src {
        char *p;                           // the frame's first point, group 0
        uint32_t start;                    // offset of the tile's first halo point
        uint32_t ok;                       // bit k: this thread's point k has a value (else it reads zero)
        int rs;                            // [TR 4] row stride, and which half the tile is
        bool odd;
    };
    auto source = [&](const TileDec &r) {
        Src s{const_cast<char *>(static_cast<const char *>(a.in)) + r.act * a.pstride,
              halo_start(r.a0, r.rs, r.cs, (uint32_t)a.pstride), 0u, r.rs,
              NPE > 0 && (walk.dd.div((uint32_t)r.y0) & 4u)};
        auto has_value = [&](int y, int x) {
            bool ok = ((unsigned)y < (unsigned)r.h) & ((unsigned)x < (unsigned)r.w);
            if constexpr (GATED) ok = ok && computed(a, r, y, x);
            return ok;
        };
#pragma unroll
        for (int k = 0; k < NPF; ++k) s.ok |= has_value(r.y0 - dd + dy[k], r.x0 - dd + dx[k]) ? 1u << k : 0u;
#pragma unroll
        for (int k = 0; k < NPE; ++k) {
            const int q = tid + k * NTH;
            int row, col;
            extra_point(q >> 2, s.odd, row, col);
            s.ok |= q < NEXTRA * 4 && has_value(r.y0 + dd * (row - 1), r.x0 + dd * (col - 1)) ? 1u << (NPF + k) : 0u;
        }
        return s;
    };
    auto load_extra = [&](const Src &s, int g) {
#pragma unroll
        for (int k = 0; k < NPE; ++k) {
            const int q = tid + k * NTH;
            int row, col;
            extra_point(q >> 2, s.odd, row, col);
            const uint32_t o = s.start + halo_point(row, col, s.rs, a.in_phase ? 1 : dd, (uint32_t)a.pstride) + (q & 3) * 16;
            pe[k] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(buf_rsrc(s.p + g * a.gstride, 0x7FFFFFFFu),
                                                                                   s.ok >> (NPF + k) & 1u ? (int)o : BUF_OOB, 0, 0));
        }
    };
    auto extra_max = [&](float m) {
#pragma unroll
        for (int k = 0; k < NPE; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) m = fmaxf(m, fabsf(pe[k][r]));
        return m;
    };
    auto load = [&](const Src &s, int g, int k) {
        return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(buf_rsrc(s.p + g * a.gstride, 0x7FFFFFFFu),
                                                                              s.ok >> k & 1u ? (int)((uint32_t)off[k] + s.start) : BUF_OOB, 0, 0));
    };
    auto largest = [&](const v4f (&p)[NPF]) {
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < NPF; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) m = fmaxf(m, fabsf(p[k][r]));
        return wave_max(extra_max(m));
    };
    auto group_max = [&](int b) {
        const v4f *p = reinterpret_cast<const v4f *>(sM + 8 * b);
        float m = fmaxf(fmaxf(p[0][0], p[0][1]), fmaxf(p[0][2], p[0][3]));
        if constexpr (TR == 8) m = fmaxf(m, fmaxf(fmaxf(p[1][0], p[1][1]), fmaxf(p[1][2], p[1][3])));
        return (uint32_t)__builtin_amdgcn_readfirstlane(__float_as_int(m));
    };

    const char *xb = sT + (row0 * PW + 16 * strip + j) * 32 + (kq & 1) * 16;
    const char *wb = sT + L::WOFF + lane * 16;

    // n: the tile in progress, n1: the next (past the last: the last again, its
    // input is loaded and not used)
    TileDec n = decode(ti), n1 = decode(ti + nslot);
    offsets(n);
    Src s1 = source(n);
#pragma unroll
    for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int k = 0; k < NPF; ++k) pf[g][k] = load(s1, g, k);
    // group 0 of the first tile into buffer 0, the maxima of groups 0 and 1
    load_extra(s1, 0);
    {
        const float m0 = largest(pf[0]);
        if (lane == 0) sM[wave] = m0;
    }
    load_extra(s1, 1);
    __syncthreads();
    uint32_t tmax = group_max(0);          // largest magnitude bits of the tile so far
    int sexp = split_exp(tmax);
    {
        const float sc = __int_as_float((127 + sexp) << 23);
#pragma unroll
        for (int k = 0; k < NPF; ++k)
            split_store(pf[0][k] * sc, L::PLANE, stage + k * (NTH / 4 * 32));
    }
    offsets(n1);
    Src s0 = s1;                           // [TR 4] the tile in progress
    s1 = source(n1);
#pragma unroll
    for (int k = 0; k < NPF; ++k) pf[0][k] = load(s1, 0, k);
    {
        const float m1 = largest(pf[1]);
        if (lane == 0) sM[8 + wave] = m1;
    }

    int buf = 0;                           // buffer of the group in progress
    for (; ti < t1; ti += nslot) {
        const TileDec n2 = decode(ti + 2 * nslot);
        const Src s2 = source(n2);
        const int Y0 = n.y0, X0 = n.x0, H = n.h, W = n.w, xo = X0 + dd * (16 * strip + j);
        v4f acc[R][NB], acx[R][NB];       // wh xh; the cross sums
#pragma unroll
        for (int y = 0; y < R; ++y)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[y][nb] = acx[y][nb] = v4f{0.f, 0.f, 0.f, 0.f};
        v4f rr[RES ? R : 1][RES ? NB : 1];
        int nexp = 0;                      // the next tile's: its group 0 is converted during this one's last
        uint32_t nmax = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            __syncthreads();   // group g staged, the other buffer free, the next group's maxima written
            // the next group's exponent: this tile's (lowered where the group
            // needs it: the sums are rescaled once this group is in them), or
            // the next tile's own
            const uint32_t gm = group_max(buf ^ 1);
            const int e = split_exp(gm);
            int se = e;
            if (g + 1 < G) {
                tmax = max(tmax, gm);
                se = min(sexp, e);
            } else {
                nexp = e;
                nmax = gm;
                offsets(n2);
            }
            const float sc = __int_as_float((127 + se) << 23);
            const Src &sl = g + 1 < G ? s1 : s2;
            const int ps = (g + 1) % 3;                  // the set of the next group, then of the group loaded
            char *sd = stage + (buf ^ 1) * L::BUF;
            const char *xp = xb + buf * L::BUF;
            if (RES && g + 1 == G) {
                __amdgpu_buffer_rsrc_t rres[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    rres[nb] = buf_rsrc(const_cast<char *>(static_cast<const char *>(a.res)) + n.act * a.pstride + nb * a.gstride,
                                        0x7FFFFFFFu);
#pragma unroll
                for (int y = 0; y < R; ++y) {
                    const bool ok = (Y0 + dd * (row0 + y) < H) & (xo < W);
                    const int o = ok ? (n.a0 + (row0 + y) * n.rs + (16 * strip + j) * n.cs) * (int)a.pstride + kq * 16 : BUF_OOB;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        rr[y][nb] = __builtin_bit_cast(
                            v4f, __builtin_amdgcn_raw_buffer_load_b128(rres[nb], o, 0, 0));
                }
            }
            // operands: x[0] rows of the three full steps (then of the second
            // closing step), x[1] of the first closing step; w alternates
            v4f x[2][R + 2][2], w[2][NB][2];
            auto read_x = [&](int set, const char *p, int rows) {
#pragma unroll
                for (int y = 0; y < rows; ++y) {
                    x[set][y][0] = *reinterpret_cast<const v4f *>(p + y * (PW * 32));
                    x[set][y][1] = *reinterpret_cast<const v4f *>(p + y * (PW * 32) + L::PLANE);
                }
            };
            auto read_w = [&](int st) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        w[st & 1][nb][h] = *reinterpret_cast<const v4f *>(wb + (((g * 5 + st) * NB + nb) * 2 + h) * 1024);
            };
            read_w(0);
            read_x(0, xp + kh * 32, R + 2);
            float mx = 0.f;
            if constexpr (NPE > 0) load_extra(g == 0 ? s0 : s1, (g + 2) % G);      // of the group after the next
#pragma unroll
            for (int c = 0; c < 15; ++c) {
                const int st = c / 3, t = c % 3;
                if (t == 0) {
                    if (st < 4) read_w(st + 1);
                    if (st == 2) read_x(1, xp + 64 + kh * (PW * 32), R);
                    if (st == 3) read_x(0, xp + 64 + 2 * (PW * 32), R);
                }
#pragma unroll
                for (int y = 0; y < R; ++y)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const v4f wv = w[st & 1][nb][t == 2], xv = x[st == 3][st < 3 ? y + st : y][t == 1];
                        v4f &d = t > 0 ? acx[y][nb] : acc[y][nb];
                        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, wv), __builtin_bit_cast(v8h, xv),
                                                                   d, 0, 0, 0);
                    }
                // between the MFMAs: the next group into the other buffer, the
                // loads that refill its registers, and the largest value of the
                // group after it
                if (c < NPF) split_store(pf[ps][c] * sc, L::PLANE, sd + c * (NTH / 4 * 32));
                if (c >= NPF && c < 2 * NPF) pf[ps][c - NPF] = load(sl, (g + 1) % G, c - NPF);
                if (c == 2 * NPF) {
#pragma unroll
                    for (int k = 0; k < NPF; ++k)
#pragma unroll
                        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, fabsf(pf[(g + 2) % 3][k][r]));
                }
                if (c == 14) {
                    mx = wave_max(extra_max(mx));
                    if (lane == 0) sM[8 * buf + wave] = mx;
                }
#pragma unroll
                for (int i = 0; i < R * NB; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // an MFMA,
                    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);     // two VALU operations
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (g + 1 < G && se < sexp) {
                const float f = __int_as_float((127 + se - sexp) << 23);
#pragma unroll
                for (int y = 0; y < R; ++y)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        acc[y][nb] *= f;
                        acx[y][nb] *= f;
                    }
                sexp = se;
            }
            buf ^= 1;
        }
        if (slow_layer | split_misfit(tmax)) {
            slow_tile<C, TR, NH>(a, n, reinterpret_cast<const float *>(static_cast<const char *>(a.wpk) + L::WBYTES), sB, sH);
        } else {
            const int osh = a.out_shift, om = (1 << osh) - 1;
            const int ohd = (H + om) >> osh, owd = (W + om) >> osh;
            __amdgpu_buffer_rsrc_t orow[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                orow[nb] = buf_rsrc(HEAD ? nullptr : static_cast<char *>(a.out) + n.act * a.pstride + nb * a.gstride,
                                    HEAD ? 0u : 0x7FFFFFFFu);
            const float ts = __int_as_float((127 - sexp) << 23);
            v4f bias[NB], scl[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                bias[nb] = *reinterpret_cast<const v4f *>(sB + nb * 16 + kq * 4);
                scl[nb] = *reinterpret_cast<const v4f *>(sS + nb * 16 + kq * 4) * ts;
            }
            auto value = [&](int y, int nb) {
                v4f v = acc[y][nb];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = fmaf(fmaf(acx[y][nb][r], 0x1p-11f, v[r]), scl[nb][r], bias[nb][r]);
                    if constexpr (RES) v[r] += rr[y][nb][r];
                }
                return relu4(v);
            };
            if constexpr (HEAD) {
                constexpr int N = head_blocks<NH, C>(R);
#pragma unroll
                for (int y0 = 0; y0 < R; y0 += N) {
                    float hh[N][NH] = {};                // head sums of this lane's channels
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        v4f vr[N];
#pragma unroll
                        for (int y = 0; y < N; ++y) vr[y] = value(y0 + y, nb);
                        head_add<NH, C>(hh, sH, nb * 16 + kq * 4, vr);
                    }
#pragma unroll
                    for (int y = 0; y < N; ++y) {
                        const int yo = Y0 + dd * (row0 + y0 + y);
                        head_store(hh[y], sH + NH * C, a.maps + NH * n.px + (int64_t)yo * W + xo, (int64_t)H * W, kq, (yo < H) & (xo < W));
                    }
                }
            } else {
#pragma unroll
                for (int y = 0; y < R; ++y) {
                    const int yo = Y0 + dd * (row0 + y);
                    const bool ok = (yo < H) & (xo < W);
                    const int opt = ((((yo & om) << osh) + (xo & om)) * ohd + (yo >> osh)) * owd + (xo >> osh);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, value(y, nb)), orow[nb],
                                                               ok ? opt * (int)a.pstride + kq * 16 : BUF_OOB, 0, 0);
                }
            }
        }
        n = n1;
        n1 = n2;
        s0 = s1;
        s1 = s2;
        sexp = nexp;
        tmax = nmax;
    }
}

// ---- packing ----
// A workgroup takes one convolution of the batch: its waves the rows' largest
// magnitudes, then each thread 16-byte pieces of the fragments, hi and lo.  (On
// the host this took 78 us a layer of 48 channels.)
struct PackBatch {
    static constexpr int MAX = 32, THREADS = 1024, ROWS = 64;
    PairJob job[MAX];
};

__global__ void __launch_bounds__(PackBatch::THREADS)
k_pack_pairs(PackBatch b)
{
    const PairJob &j = b.job[blockIdx.x];
    __shared__ float up[PackBatch::ROWS];
    __shared__ int misfit;
    const int tid = threadIdx.x, lane = tid & 63, row = j.cin * j.taps;
    if (tid == 0) misfit = 0;
    __syncthreads();
    for (int oc = tid >> 6; oc < j.cout; oc += PackBatch::THREADS / 64) {
        const float *w = j.w + (size_t)oc * j.ld * j.taps;
        uint32_t mb = 0;                               // magnitudes order as integers, NaNs last
        for (int k = lane; k < row; k += 64) mb = max(mb, __float_as_uint(w[k]) & 0x7FFFFFFFu);
#pragma unroll
        for (int d = 32; d; d >>= 1) mb = max(mb, (uint32_t)__shfl_xor((int)mb, d));
        const int e = (int)(mb >> 23) - 127;           // the largest weight lies in [2^e, 2^(e + 1))
        const int s = mb ? min(60, max(-60, 14 - e)) : 0;
        if (lane == 0) {
            up[oc] = __int_as_float((127 + s) << 23);
            j.scale[oc] = __int_as_float((127 - s) << 23);
            if (mb && (e < -60 || e >= 75)) misfit = 1;
        }
    }
    __syncthreads();
    if (misfit)
        for (int oc = tid; oc < j.cout; oc += PackBatch::THREADS) j.scale[oc] = 0.f;
    if (j.raw)
        for (int k = tid; k < j.cout * row; k += PackBatch::THREADS) j.raw[k] = j.w[k];      // (ld = cin)
    const int NB = j.cout / 16, NS = pair_steps(j.taps, j.group), CH8 = j.group / 8, FULL = 3 * CH8 / 4;
    const int pieces = j.cin / j.group * NS * NB * 64;
    uint4 *dst = static_cast<uint4 *>(j.dst);
    for (int p = tid; p < pieces; p += PackBatch::THREADS) {
        const int i = p & 15, kq = p >> 4 & 3, nb = (p >> 6) % NB, st = (p >> 6) / NB;
        const int g = st / NS, sg = st - g * NS, oc = nb * 16 + i;
        // the lanes' tap (-1: zero weights) and 8 channels: steps of a tap row u take
        // chunks of 8 channels, tap column major, four at a time; the closing two the
        // chunks left over (SPlan).  1x1: the centre half of the second closing step.
        int tap, c0 = g * j.group;
        if (j.taps == 1) {
            tap = kq < 2 ? -1 : 0;
            c0 += (kq & 1) * 8;
        } else {
            const bool closing = sg >= 3 * FULL;
            const int u = !closing ? sg % 3 : sg == 3 * FULL ? kq >> 1 : kq < 2 ? 2 : 3;
            const int chunk = closing ? 4 * FULL + (kq & 1) : 4 * (sg / 3) + kq;
            tap = u < 3 ? 3 * u + chunk / CH8 : -1;
            c0 += chunk % CH8 * 8;
        }
        uint32_t hi[4] = {}, lo[4] = {};
        if (tap >= 0 && !misfit) {
            const float *w = j.w + ((size_t)oc * j.ld + c0) * j.taps + tap;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a = w[2 * e * j.taps] * up[oc], c = w[(2 * e + 1) * j.taps] * up[oc];
                const float ah = (float)(_Float16)a, ch = (float)(_Float16)c;
                hi[e] = pack_h2(ah, ch);
                lo[e] = pack_h2((a - ah) * 2048.f, (c - ch) * 2048.f);
            }
        }
        uint4 *f = dst + (size_t)(st * NB + nb) * 128 + kq * 16 + i;
        f[0] = uint4{hi[0], hi[1], hi[2], hi[3]};
        f[64] = uint4{lo[0], lo[1], lo[2], lo[3]};
    }
}

// ------------------------------------------------------------- launchers
template <int C, int TR> constexpr int split_threads() { return C == 48 ? TR * 64 : NTH; }

template <int C, int TR, bool RES, int NH, bool GATED = false>
auto kernel_of()
{
    if constexpr (C == 48) return k_pipe<C, TR, RES, NH, GATED>;
    else return k_split<C, TR, RES, NH, GATED>;
}

template <int C, int TR, bool RES, int NH, bool GATED>
hipError_t launch_g(const ConvArgs &a, const Geometry &g, int grid, hipStream_t s)
{
    using L = std::conditional_t<C == 48, PLds<C, TR, (NH > 5 ? NH : 5)>, SLds<C, TR, (NH > 5 ? NH : 5)>>;
    static_assert(L::FITS, "LDS of the split kernel");
    auto kern = kernel_of<C, TR, RES, NH, GATED>();
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, L::TOTAL);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(split_threads<C, TR>()), L::TOTAL, s, a, g);
    return hipGetLastError();
}

// (GATED: the kernels that leave out points no layer computed; the test in the
// others' load paths costs 2 to 4%, unused)
template <int C, int TR, bool RES, int NH>
hipError_t launch_k(const ConvArgs &a, const Geometry &g, int grid, hipStream_t s)
{
    return a.keep ? launch_g<C, TR, RES, NH, true>(a, g, grid, s) : launch_g<C, TR, RES, NH, false>(a, g, grid, s);
}

template <int C, int TR>
hipError_t launch_tr(const ConvArgs &a, const Geometry &g, int grid, hipStream_t s)
{
    if (a.head) return a.nh == 10 ? launch_k<C, TR, true, 10>(a, g, grid, s) : launch_k<C, TR, true, 5>(a, g, grid, s);
    if (a.res) return launch_k<C, TR, true, 0>(a, g, grid, s);
    return launch_k<C, TR, false, 0>(a, g, grid, s);
}

template <int C, int TR>
int blocks_per_cu()
{
    int nb = 0;
    auto kern = kernel_of<C, TR, true, 0>();
    constexpr size_t sh = std::conditional_t<C == 48, PLds<C, TR, 5>, SLds<C, TR, 5>>::TOTAL;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, split_threads<C, TR>(), sh) != hipSuccess) nb = 1;
    return nb > 0 ? nb : 1;
}

}  // namespace

bool split_takes(int C, int precision) { return C <= 48 && precision == DL_FP32; }

size_t split_packed_bytes(int C) { return pair_packed_bytes(C, C, 9, split_pack_group(C)) + (size_t)9 * C * C * 4; }

hipError_t launch_pack_pairs(const PairJob *jobs, int n, hipStream_t s)
{
    for (int i = 0; i < n; i += PackBatch::MAX) {
        PackBatch b{};
        const int m = std::min(n - i, PackBatch::MAX);
        for (int k = 0; k < m; ++k) {
            const PairJob &j = b.job[k] = jobs[i + k];
            if (j.cout % 16 || j.cout > PackBatch::ROWS || j.group % 16 || j.cin % j.group || j.ld < j.cin ||
                !(j.taps == 9 ? j.group <= 32 : j.taps == 1 && j.group == 16))
                return hipErrorInvalidValue;
        }
        hipLaunchKernelGGL(k_pack_pairs, dim3(m), dim3(PackBatch::THREADS), 0, s, b);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

int split_max_grid(int C, int tr, int ncu)
{
    switch (C) {
    case 16: return ncu * (tr == 4 ? blocks_per_cu<16, 4>() : blocks_per_cu<16, 8>());
    case 32: return ncu * (tr == 4 ? blocks_per_cu<32, 4>() : blocks_per_cu<32, 8>());
    default: return ncu * (tr == 4 ? blocks_per_cu<48, 4>() : blocks_per_cu<48, 8>());
    }
}

hipError_t launch_split(int C, const ConvArgs &a, const Geometry &g, int grid, hipStream_t s)
{
    switch (C) {
    case 16: return a.tr == 4 ? launch_tr<16, 4>(a, g, grid, s) : launch_tr<16, 8>(a, g, grid, s);
    case 32: return a.tr == 4 ? launch_tr<32, 4>(a, g, grid, s) : launch_tr<32, 8>(a, g, grid, s);
    case 48: return a.tr == 4 ? launch_tr<48, 4>(a, g, grid, s) : launch_tr<48, 8>(a, g, grid, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dloc
