// Inference of the dense-connection networks' layers (paper Sec. 3.2, 3.2.1,
// 4.1.2) on the FP16 matrix cores: 3x3 dilated convolutions over a growing
// concatenation, with the block's 1x1 transition and the 1x1 head fused into
// its last layer, and the U-Net's convolutions (gfx950).
//
// Operands, products, scaling (22 bits of what is within 2^28 of a tile's or a
// row's largest) and the plain-FP32 tile of values outside the FP16 halves' range
// are those of kernels_split.hip; so is the walk over K in
// groups of 16 channels (k_pipe), here over as many groups as the
// concatenation has: every group's tile goes through one of two LDS buffers
// while the next one is converted into the other and the loads of the two
// after that are in flight.  The transition's products of a group ride on the
// closing step's fragment, whose upper lane groups hold the centre tap; its
// last channels, the layer's own outputs, and the head are FP32 MFMAs on the
// accumulators' values (as k_dconv, kernels_dense.hip).
//
// Activations lie in planes of 16 channels, 64 bytes per point: a group's tile
// row is one contiguous run, and a layer appends planes to the concatenation.
// (In NHWC a point of 96 channels is 384 bytes, of which a layer of 48 read two
// and a half 128-byte lines to use one and a half.)  Within a plane a block's
// points lie in the phase layout of its dilation (phase_point).
//
// What bounds it: the issue slots of a step whose 16 outputs leave few MFMAs
// (27 a wave and group of 64 points) beside the conversion of the group's tile,
// then HBM (64 bytes a point and group read, 64 written).  Net D at 4 x 2048^2,
// FP32 matrix cores -> FP16 pairs: a layer 2.09 -> 1.07 ms (4.4 TB/s), a last
// layer with its transition 3.98 -> 2.50 ms, with the head 4.27 -> 2.78 ms.
#include <algorithm>

#include "conv_common.h"
#include "split_common.h"

namespace dloc {

namespace {

constexpr int TR = 8, TC = 32, PW = TC + 2, NTH = 512, R = 2;   // eight waves of 2 x 16 points
constexpr int NPT = (TR + 2) * PW, NQ = NPT * 4, NPF = (NQ + NTH - 1) / NTH;
constexpr int PLANE = NPF * NTH / 4 * 32, BUF = 2 * PLANE;    // (room for the chunks past the last point)

// LDS: two group buffers, the constants, then the weights: of every group when
// they fit (resident), else of two groups in turn
template <int NB, int NT, int FUSE> struct DL {
    static constexpr bool TRN = FUSE == 1 || FUSE == 2, HD = FUSE >= 2;
    static constexpr int HK = FUSE == 3 ? NB : NT;                 // head K groups
    static constexpr int WL = 5 * NB * 2048;                       // one group's layer fragments
    static constexpr int WG = WL + (TRN ? NT * 2048 : 0);          // + its transition fragments
    // workgroups that share a CU and hide each other's conversion and epilogue:
    // two where the accumulators leave a wave's needs at 128 registers (with two
    // sets of loads in flight each), else one with three sets.  (Four waves of
    // four rows in 256 registers spill with the transition's accumulators.)
    static constexpr int WGS = NB == 1 && !TRN ? 2 : 1, SETS = WGS == 2 ? 2 : 3;
    static constexpr int NWF = (WG / 16 + NTH - 1) / NTH;
    static constexpr int WTL = BUF * 2;                            // transition of the layer's outputs (FP32)
    static constexpr int WH = WTL + (TRN ? NB * NT * 1024 : 0);    // head (FP32)
    static constexpr int BO = WH + (HD ? HK * 1024 : 0);           // bias, scale [16 NB]; transition's [16 NT]; head's [16]
    static constexpr int MO = BO + (2 * NB * 16 + (TRN ? 2 * NT * 16 : 0) + (HD ? 16 : 0)) * 4;   // maxima [2][8]
    static constexpr int QO = MO + 64;                             // claimed tiles [8]
    static constexpr int TO = QO + 32;                             // decoded tiles [8]
    static constexpr int W = TO + 8 * 64;
    static constexpr int bytes(int ngroups, bool res) { return W + (res ? ngroups : 2) * WG; }
};

// One tile in plain FP32 (see split_misfit): a thread per output point.
template <int NB, int NT, int FUSE>
__device__ __forceinline__ void dslow_tile(const DensePipeArgs &a, const TileDec &n)
{
    using L = DL<NB, NT, FUSE>;
    const int row = threadIdx.x / TC, col = threadIdx.x % TC, cin = a.ngroups * 16;
    const int yo = n.y0 + a.d * row, xo = n.x0 + a.d * col;
    if (row >= TR || yo >= n.h || xo >= n.w) return;
    const int64_t pt = n.act + n.a0 + (int64_t)row * n.rs + col * n.cs;
    const int64_t tpt = n.act + phase_point(n.h, n.w, a.out_shift, yo, xo);
    auto in = [&](int64_t p, int c) { return a.in[(c >> 4) * a.igs + p * 16 + (c & 15)]; };
    float t[L::HK * 16] = {};            // the transition's outputs, or (FUSE 3) the layer's
    const int ct = cin + NB * 16;
    if constexpr (L::TRN)
#pragma unroll 1
        for (int c = 0; c < cin; ++c) {
            const float x = in(pt, c);
#pragma unroll
            for (int k = 0; k < NT * 16; ++k) t[k] = fmaf(a.traw[k * ct + c], x, t[k]);
        }
#pragma unroll 1
    for (int oc = 0; oc < NB * 16; ++oc) {
        float s = 0.f;
#pragma unroll 1
        for (int tap = 0; tap < 9; ++tap) {
            const int yy = yo + a.d * (tap / 3 - 1), xx = xo + a.d * (tap % 3 - 1);
            if ((unsigned)yy >= (unsigned)n.h || (unsigned)xx >= (unsigned)n.w) continue;
            const int64_t p = pt + (int64_t)(tap / 3 - 1) * n.rs + (tap % 3 - 1) * n.cs;
#pragma unroll 1
            for (int c = 0; c < cin; ++c) s = fmaf(a.raw[((int64_t)oc * cin + c) * 9 + tap], in(p, c), s);
        }
        s = fmaxf(s + a.bias[oc], 0.f);
        if constexpr (FUSE == 0) a.out[(oc >> 4) * a.ogs + pt * 16 + (oc & 15)] = s;
        if constexpr (L::TRN)
#pragma unroll
            for (int k = 0; k < NT * 16; ++k) t[k] = fmaf(a.traw[k * ct + cin + oc], s, t[k]);
        if constexpr (FUSE == 3)
#pragma unroll
            for (int k = 0; k < NB * 16; ++k) t[k] = k == oc ? s : t[k];
    }
    if constexpr (L::TRN)
#pragma unroll
        for (int k = 0; k < NT * 16; ++k) {
            t[k] = fmaxf(t[k] + a.bt[k], 0.f);
            if constexpr (FUSE == 1) a.tout[(k >> 4) * a.tgs + tpt * 16 + (k & 15)] = t[k];
        }
    if constexpr (L::HD)
#pragma unroll 1
        for (int q = 0; q < a.nh; ++q) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < L::HK * 16; ++k) s = fmaf(a.hraw[q * L::HK * 16 + k], t[k], s);
            a.maps[a.nh * n.px + ((int64_t)q * n.h + yo) * n.w + xo] = s + a.bh[q];
        }
}

__device__ const v4f zeros = {0.f, 0.f, 0.f, 0.f};
typedef __attribute__((address_space(1))) v4f global_v4f;    // (a generic pointer would make the loads flat)

// FUSE: 0 the layer alone; 1 + the block's 1x1 transition; 2 + transition +
// head; 3 + head (on the layer's own outputs).  QUEUE: tiles claimed from
// atomic queues instead of the static ranges per XCD.
template <int NB, int NT, int FUSE, bool QUEUE>
__global__ void __launch_bounds__(NTH, (2 * DL<NB, NT, FUSE>::WGS))
k_dpipe(DensePipeArgs a, Geometry geo)
{
    using L = DL<NB, NT, FUSE>;
    constexpr bool TRN = L::TRN, HD = L::HD;
    constexpr int SETS = L::SETS;
    extern __shared__ v4f smem[];
    char *sT = reinterpret_cast<char *>(smem);
    const v4f *sWTL = reinterpret_cast<const v4f *>(sT + L::WTL), *sWH = reinterpret_cast<const v4f *>(sT + L::WH);
    float *sB = reinterpret_cast<float *>(sT + L::BO), *sS = sB + NB * 16;
    float *sBT = sS + NB * 16, *sST = sBT + NT * 16, *sBH = sBT + (TRN ? 2 * NT * 16 : 0);
    float *sM = reinterpret_cast<float *>(sT + L::MO);
    int *sQ = reinterpret_cast<int *>(sT + L::QO), *sD = reinterpret_cast<int *>(sT + L::TO);
    v4f *sW = reinterpret_cast<v4f *>(sT + L::W);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kq = lane >> 4, kh = kq >> 1;
    const int strip = wave & 1, row0 = (wave >> 1) * R;
    const int dd = a.d, blk = a.blk, G = a.ngroups;
    const bool res = a.wres;
    const v4f *gw = static_cast<const v4f *>(a.w), *gt = static_cast<const v4f *>(a.wt);
    // 16-byte piece i of group g's weights: the layer's fragments, then the transition's
    auto wpiece = [&](int g, int i) {
        if constexpr (TRN) return i < L::WL / 16 ? gw[g * (L::WL / 16) + i] : gt[g * (NT * 128) + i - L::WL / 16];
        else return gw[g * (L::WL / 16) + i];
    };
    if (res)
        for (int g = 0; g < G; ++g)
            for (int i = tid; i < L::WG / 16; i += NTH) sW[g * (L::WG / 16) + i] = wpiece(g, i);
    for (int i = tid; i < NB * 16; i += NTH) {
        sB[i] = a.bias[i];
        sS[i] = a.scale[i];
    }
    bool slow_layer = ld_const(a.scale) == 0.f;
    if constexpr (TRN) {
        for (int i = tid; i < NB * NT * 64; i += NTH) const_cast<v4f *>(sWTL)[i] = reinterpret_cast<const v4f *>(a.wtl)[i];
        for (int i = tid; i < NT * 16; i += NTH) {
            sBT[i] = a.bt[i];
            sST[i] = a.st[i];
        }
        slow_layer |= ld_const(a.st) == 0.f;
    }
    if constexpr (HD) {
        for (int i = tid; i < L::HK * 64; i += NTH) const_cast<v4f *>(sWH)[i] = reinterpret_cast<const v4f *>(a.wh)[i];
        for (int i = tid; i < 16; i += NTH) sBH[i] = i < a.nh ? a.bh[i] : 0.f;
    }

    const int64_t T = geo.dyn ? ld_const(geo.dyn + DYN_TILES + blk) : geo.tiles[blk];
    const int nfr = geo.dyn ? (int)ld_const(geo.dyn + DYN_NF) : geo.nf;
    const int xcd = blockIdx.x % NXCD, slot = blockIdx.x / NXCD, nslot = gridDim.x / NXCD;
    const int64_t chunk = (T + NXCD - 1) / NXCD;
    const int64_t t0 = (int64_t)xcd * chunk, t1 = min(T, t0 + chunk);
    // The workgroup's k-th tile: t0 + slot + k nslot of the XCD's range, or
    // (QUEUE) the k-th it claimed from the XCD's queue (queue_mode 1) or the one
    // queue over all tiles (2); the claims are made one tile ahead of their use
    // and pass through LDS.  A tile at or past `end` does not exist.
    const bool one = QUEUE && a.queue_mode == 2;
    const int64_t qb = one ? 0 : t0, end = one ? T : t1;
    auto claim = [&](int k) {
        if (QUEUE && tid == 0) sQ[k & 7] = (int)min<uint32_t>(atomicAdd(a.queue + (one ? 0 : xcd), 1u), 0x7FFFFFFFu);
    };
    auto tile_id = [&](int k) -> int64_t {
        if constexpr (QUEUE) return qb + (uint32_t)__builtin_amdgcn_readfirstlane(sQ[k & 7]);
        else return t0 + slot + (int64_t)k * nslot;
    };
    claim(0);
    claim(1);
    __syncthreads();                     // claims and constants are in LDS
    if (tile_id(0) >= end) return;       // uniform over the workgroup

    // staging: chunk k of a thread is 4 channels of one point of the group's tile
    v4f pf[SETS][NPF];                   // the next item and the one(s) after it
    int off[NPF];                        // from the tile's first point, in 16 bytes (fits for points of the frame)
    int dy[NPF], dx[NPF], off_rs = -1;
    char *const stage = sT + (tid >> 2) * 32 + (tid & 3) * 8;
#pragma unroll
    for (int k = 0; k < NPF; ++k) {
        const int q = tid + k * NTH, pt = q >> 2;
        dy[k] = q < NQ ? dd * (pt / PW) : 1 << 30;       // past the last chunk: off every frame
        dx[k] = dd * (pt - pt / PW * PW);
    }
    // the load cursor: the tile and group whose input is loaded next (past the
    // last tile, the last one over again: loaded and not used)
    TileWalk walk;
    int lk = -1, lg = G - 1, ly = 0, lx = 0, lh = 0, lw = 0;
    const v4f *lp = nullptr;             // the tile's first point in plane 0
    // The cursor moves on by one group.  A new tile (whose claim was published
    // before the last barrier) is decoded once and handed to the item that will
    // need its place through LDS.
    auto advance = [&]() {
        if (++lg < G) return;
        lg = 0;
        const int64_t t = tile_id(lk + 1);
        if (t >= end) return;
        ++lk;
        TileDec r = walk.tile(a, geo, nfr, TR, TC, t);
        r.a0 = (int)phase_point(r.h, r.w, a.in_shift, r.y0, r.x0);
        if (a.in_shift) {
            r.rs = (r.w - (r.x0 & (dd - 1)) + dd - 1) >> a.in_shift;     // the sub-image's columns
            r.cs = 1;
        }
        if (wave == 0) publish_tile(sD + (lk & 7) * 16, lane, r);
        claim(lk + 2);
        ly = r.y0 - dd;
        lx = r.x0 - dd;
        lh = r.h;
        lw = r.w;
        lp = reinterpret_cast<const v4f *>(a.in) + (r.act + r.a0) * 4;
        if (r.rs != off_rs) {
            off_rs = r.rs;
#pragma unroll
            for (int k = 0; k < NPF; ++k) {
                const int q = tid + k * NTH, pt = q >> 2;
                off[k] = (int)((uint32_t)(pt / PW - 1) * (uint32_t)r.rs + (uint32_t)((pt - pt / PW * PW - 1) * r.cs)) * 4 + (q & 3);
            }
        }
    };
    const int64_t gs4 = a.igs / 4;
    auto load = [&](v4f (&p)[NPF]) {     // points off the frame read zeros
        const v4f *gp = lp + lg * gs4;
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const bool ok = ((unsigned)(ly + dy[k]) < (unsigned)lh) & ((unsigned)(lx + dx[k]) < (unsigned)lw);
            p[k] = *(ok ? (const global_v4f *)(gp + off[k]) : (const global_v4f *)&zeros);
        }
    };
    auto largest = [&](const v4f (&p)[NPF]) {
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < NPF; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) m = fmaxf(m, fabsf(p[k][r]));
        return wave_max(m);
    };
    auto group_max = [&](int b) {
        const v4f *p = reinterpret_cast<const v4f *>(sM + 8 * b);
        float m = fmaxf(fmaxf(p[0][0], p[0][1]), fmaxf(p[0][2], p[0][3]));
        m = fmaxf(m, fmaxf(fmaxf(p[1][0], p[1][1]), fmaxf(p[1][2], p[1][3])));
        return (uint32_t)__builtin_amdgcn_readfirstlane(__float_as_int(m));
    };
    v4f wf[L::NWF];
    auto load_w = [&](int g) {           // a group's weights (not resident) into registers
        if (!res)
#pragma unroll
            for (int k = 0; k < L::NWF; ++k) {
                wf[k] = wpiece(g, min(tid + k * NTH, L::WG / 16 - 1));
            }
    };
    auto store_w = [&](int b) {
        if (!res)
#pragma unroll
            for (int k = 0; k < L::NWF; ++k) {
                sW[b * (L::WG / 16) + min(tid + k * NTH, L::WG / 16 - 1)] = wf[k];
            }
    };

    // fill: item 0 converted into buffer 0, items 1 .. SETS in registers, the
    // maxima of items 0 and 1
    v4f p0[NPF];
    advance();
    load(p0);
    __syncthreads();                     // (each advance needs the claim of an earlier one published)
    advance();
    load(pf[0]);
    __syncthreads();
    advance();
    load(pf[1]);
    if constexpr (SETS == 3) {
        __syncthreads();
        advance();
        load(pf[2]);
    }
    load_w(0);
    {
        const float m0 = largest(p0), m1 = largest(pf[0]);
        if (lane == 0) {
            sM[wave] = m0;
            sM[8 + wave] = m1;
        }
    }
    __syncthreads();
    uint32_t tmax = group_max(0);        // largest magnitude bits of the tile so far
    int sexp = split_exp(tmax);
    {
        const float sc = __int_as_float((127 + sexp) << 23);
#pragma unroll
        for (int k = 0; k < NPF; ++k) split_store(p0[k] * sc, PLANE, stage + k * (NTH / 4 * 32));
    }
    store_w(0);
    load_w(G > 1 ? 1 : 0);

    const char *const xb = sT + (row0 * PW + 16 * strip + j) * 32 + (kq & 1) * 16;
    int g = 0, kc = 0, buf = 0;          // group and tile in progress, their buffer
    v4f acc[R][NB], acx[R][NB], at[R][TRN ? NT : 1], atx[R][TRN ? NT : 1];
    auto clear = [&]() {
#pragma unroll
        for (int y = 0; y < R; ++y) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[y][nb] = acx[y][nb] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int nt = 0; nt < (TRN ? NT : 1); ++nt) at[y][nt] = atx[y][nt] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    };
    clear();

    // one item, the MFMAs of group g, with the next item's registers, and those
    // of the one after it; false after the last tile.  (A copy per register set:
    // moving a set would wait for its loads.)
    auto item = [&](v4f (&pn)[NPF], v4f (&pm)[NPF]) -> bool {
        __syncthreads();   // this group staged, the other buffer free, the next item's maxima written
        const bool more = g + 1 < G;
        const int gn = more ? g + 1 : 0;
        const uint32_t gm = group_max(buf ^ 1);
        const int e = split_exp(gm), se = more ? min(sexp, e) : e;
        if (more) tmax = max(tmax, gm);
        const char *xp = xb + buf * BUF;
        const char *wb = reinterpret_cast<const char *>(sW) + (res ? g : buf) * L::WG + lane * 16;
        // the next item into the other buffer, the loads that refill its registers
        {
            const float sc = __int_as_float((127 + se) << 23);
            char *d = stage + (buf ^ 1) * BUF;
#pragma unroll
            for (int k = 0; k < NPF; ++k) split_store(pn[k] * sc, PLANE, d + k * (NTH / 4 * 32));
            store_w(buf ^ 1);
            load_w(gn + 1 < G ? gn + 1 : 0);
            advance();
            load(pn);
        }

        auto mm = [&](const v4f &wv, const v4f &xv, v4f &d) {
            d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, wv), __builtin_bit_cast(v8h, xv), d, 0, 0, 0);
        };
        // full steps: taps v = 0 (lane groups 0, 1) and 1 of tap row u = st;
        // closing steps, v = 2: rows u = 0 and 1, then row u = 2 beside the
        // centre tap (which the transition takes; the layer's weights there are
        // zero).  Each with the hi halves of x, then the lo halves.
        const char *xs[3] = {xp + kh * 32, xp + 64 + kh * (PW * 32), xp + (kh ? PW * 32 + 32 : 2 * PW * 32 + 64)};
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4f x[R + 2];
#pragma unroll
                for (int y = 0; y < (s == 0 ? R + 2 : R); ++y)
                    x[y] = *reinterpret_cast<const v4f *>(xs[s] + y * (PW * 32) + h * PLANE);
#pragma unroll
                for (int u = 0; u < (s == 0 ? 3 : 1); ++u)
#pragma unroll
                    for (int wh = 0; wh < 2 - h; ++wh)       // wh xh, wl xh; wh xl
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            const int st = s == 0 ? u : s + 2;
                            const v4f wv = *reinterpret_cast<const v4f *>(wb + ((st * NB + nb) * 2 + wh) * 1024);
#pragma unroll
                            for (int y = 0; y < R; ++y) mm(wv, x[y + u], h + wh ? acx[y][nb] : acc[y][nb]);
                        }
                if constexpr (TRN)
                    if (s == 2)
#pragma unroll
                        for (int wh = 0; wh < 2 - h; ++wh)
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt) {
                                const v4f wv = *reinterpret_cast<const v4f *>(wb + L::WL + (nt * 2 + wh) * 1024);
#pragma unroll
                                for (int y = 0; y < R; ++y) mm(wv, x[y], h + wh ? atx[y][nt] : at[y][nt]);
                            }
            }
        {
            const float m = largest(pm);             // of the item after the next
            if (lane == 0) sM[8 * buf + wave] = m;
        }
        buf ^= 1;
        if (more) {
            if (se < sexp) {                         // the tile goes on under a lower exponent
                const float f = __int_as_float((127 + se - sexp) << 23);
#pragma unroll
                for (int y = 0; y < R; ++y) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        acc[y][nb] *= f;
                        acx[y][nb] *= f;
                    }
                    if constexpr (TRN)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            at[y][nt] *= f;
                            atx[y][nt] *= f;
                        }
                }
                sexp = se;
            }
            ++g;
            return true;
        }

        // the tile is complete
        const TileDec n = pickup_tile(sD + (kc & 7) * 16);
        if (slow_layer | split_misfit(tmax)) {
            dslow_tile<NB, NT, FUSE>(a, n);
        } else {
            // lane (j, kq) holds output channels 16 nb + 4 kq + r of pixel j
            const float ts = __int_as_float((127 - sexp) << 23);
            const int xo = n.x0 + dd * (16 * strip + j);
#pragma unroll
            for (int y = 0; y < R; ++y) {
                const int yo = n.y0 + dd * (row0 + y);
                const bool inside = (yo < n.h) & (xo < n.w);
                const int64_t pt = (n.act + n.a0 + (int64_t)(row0 + y) * n.rs + (16 * strip + j) * n.cs) * 16 + kq * 4;
                v4f o[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const v4f sl = *reinterpret_cast<const v4f *>(sS + nb * 16 + kq * 4) * ts;
                    const v4f bs = *reinterpret_cast<const v4f *>(sB + nb * 16 + kq * 4);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        o[nb][r] = fmaxf(fmaf(fmaf(acx[y][nb][r], 0x1p-11f, acc[y][nb][r]), sl[r], bs[r]), 0.f);
                }
                if constexpr (FUSE == 0) {
                    if (inside)
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<v4f *>(a.out + nb * a.ogs + pt) = o[nb];
                }
                v4f hin[L::HK];                      // the head's input: transition or layer outputs
                if constexpr (TRN) {
                    const int64_t tpt = (n.act + phase_point(n.h, n.w, a.out_shift, yo, xo)) * 16 + kq * 4;
                    // the layer's outputs are the transition's last K groups: lane (j, kq)
                    // element s is channel 4 kq + s of pixel j, the FP32 MFMA's B operand
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const v4f sl = *reinterpret_cast<const v4f *>(sST + nt * 16 + kq * 4) * ts;
                        const v4f bs = *reinterpret_cast<const v4f *>(sBT + nt * 16 + kq * 4);
                        v4f t;
#pragma unroll
                        for (int r = 0; r < 4; ++r) t[r] = fmaf(fmaf(atx[y][nt][r], 0x1p-11f, at[y][nt][r]), sl[r], bs[r]);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            const v4f aw = sWTL[(nb * NT + nt) * 64 + lane];
#pragma unroll
                            for (int s = 0; s < 4; ++s) t = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[s], o[nb][s], t, 0, 0, 0);
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) t[r] = fmaxf(t[r], 0.f);
                        if constexpr (FUSE == 1) {
                            if (inside) *reinterpret_cast<v4f *>(a.tout + nt * a.tgs + tpt) = t;
                        } else {
                            hin[nt] = t;
                        }
                    }
                } else if constexpr (HD) {
#pragma unroll
                    for (int k = 0; k < L::HK; ++k) hin[k] = o[k];
                }
                if constexpr (HD) {
                    // head: outputs q = 4 kq + r of pixel j
                    v4f hq = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < L::HK; ++k) {
                        const v4f aw = sWH[k * 64 + lane];
#pragma unroll
                        for (int s = 0; s < 4; ++s) hq = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[s], hin[k][s], hq, 0, 0, 0);
                    }
                    if (inside) {
                        const int64_t plane = (int64_t)n.h * n.w;
                        float *mp = a.maps + a.nh * n.px + (int64_t)yo * n.w + xo;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int q = 4 * kq + r;
                            if (q < a.nh) mp[q * plane] = hq[r] + sBH[q];
                        }
                    }
                }
            }
        }
        g = 0;
        sexp = e;
        tmax = gm;
        if (tile_id(++kc) >= end) return false;
        clear();
        return true;
    };
    if constexpr (SETS == 3)
        while (item(pf[0], pf[1]) && item(pf[1], pf[2]) && item(pf[2], pf[0])) {}
    else
        while (item(pf[0], pf[1]) && item(pf[1], pf[0])) {}
}

template <int NB, int NT, int FUSE, bool QUEUE>
hipError_t launch_q(DensePipeArgs a, const Geometry &g, int ncu, hipStream_t s)
{
    using L = DL<NB, NT, FUSE>;
    auto kern = k_dpipe<NB, NT, FUSE, QUEUE>;
    static_assert(L::bytes(0, false) <= 160 * 1024, "LDS of the dense kernel");
    a.wres = L::bytes(a.ngroups, true) <= 160 * 1024 / L::WGS;
    const int bytes = L::bytes(a.ngroups, a.wres);
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr = true;
    }
    int per = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, NTH, bytes) != hipSuccess || per < 1) per = 1;
    const int64_t tiles = g.dyn ? (int64_t)1 << 40 : g.tiles[a.blk];
    int grid = (int)std::min<int64_t>(tiles, (int64_t)per * ncu);
    grid = std::max(NXCD, grid / NXCD * NXCD);
    Geometry gg = g;
    gg.minor_blk = -1;                   // tiles in phase-major order, strips of 8 regions
    gg.strip = 8;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NTH), bytes, s, a, gg);
    return hipGetLastError();
}

template <int NB, int NT, int FUSE>
hipError_t launch_t(const DensePipeArgs &a, const Geometry &g, int ncu, hipStream_t s)
{
    return a.queue ? launch_q<NB, NT, FUSE, true>(a, g, ncu, s) : launch_q<NB, NT, FUSE, false>(a, g, ncu, s);
}

template <int NB, int FUSE>
hipError_t launch_nt(int nt, const DensePipeArgs &a, const Geometry &g, int ncu, hipStream_t s)
{
    if (nt == 1) return launch_t<NB, 1, FUSE>(a, g, ncu, s);
    if (nt == 2) return launch_t<NB, 2, FUSE>(a, g, ncu, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_dpipe(int nb_out, int fuse, int nt, const DensePipeArgs &a, const Geometry &g, int ncu, hipStream_t s)
{
    if (a.nh > 16 || (nb_out != 1 && nb_out != 2)) return hipErrorInvalidValue;
    switch (fuse) {
    case 0: return nb_out == 1 ? launch_t<1, 1, 0>(a, g, ncu, s) : launch_t<2, 1, 0>(a, g, ncu, s);
    case 1: return nb_out == 1 ? launch_nt<1, 1>(nt, a, g, ncu, s) : launch_nt<2, 1>(nt, a, g, ncu, s);
    case 2: return nb_out == 1 ? launch_nt<1, 2>(nt, a, g, ncu, s) : launch_nt<2, 2>(nt, a, g, ncu, s);
    case 3: return nb_out == 1 ? launch_t<1, 1, 3>(a, g, ncu, s) : launch_t<2, 1, 3>(a, g, ncu, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dloc
