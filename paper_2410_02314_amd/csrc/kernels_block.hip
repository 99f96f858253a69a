// A residual block's two 3x3 convolutions in one kernel, BF16 (gfx950):
//     t = relu(conv1(x) + b1),  y = relu(x + conv2(t) + b2)
// (paper Sec. 3.2.1), the last block with the fused 1x1 head.  t never leaves
// the CU.  As two layers (k_conv) a block moves x, t, t, x and y through HBM at
// 0.84 of the copy rate, and nothing but fewer bytes makes it faster; here it
// moves x and y, and computes t again on the rim of each tile (1.29 times its
// points).  Products, their order and every rounding are those of the two layers,
// so the maps are the same bit for bit.
//
// A workgroup (8 waves) takes the conv layers' phase tiles of 8 x 64 lattice
// points (conv_tiles, decode_tile): x on 12 x 68 points is staged in LDS, t on
// 10 x 66 points is computed in blocks of 16 consecutive points (42 blocks over
// 8 waves, their accumulators in registers), written over x after a barrier, zero
// off the frame, and wave w computes row w of y from it.  Both weights stay in
// LDS; at 48 channels that is all of it but 72 bytes, the padding of the last K
// step left out.  The next tile's x is loaded into registers while this tile
// computes.
//
// What bounds it: the phases between the barriers, which one workgroup per CU
// does not overlap -- at 32 channels a fifth of the time is MFMAs (1.2 times the
// two layers'), as much VALU.  Net A, 4 x 512^2: a block 80 -> 70 us.
#include "conv_common.h"

namespace dloc {

namespace {

constexpr int TR = 8, TC = 64, NTH = TR * 64, PB = TC / 16;
constexpr int XW = TC + 4, NX = (TR + 4) * XW, MW = TC + 2, NM = (TR + 2) * MW;
constexpr int NBLK = (NM + 15) / 16, LO = NBLK / 8, HI = (NBLK + 7) / 8;    // blocks of t: LO or HI a wave

template <int C, int NH> struct BL {
    static constexpr int NB = C / 16, CH8 = C / 8, NCH = 9 * CH8, NIT = (NCH + 3) / 4, REM = NCH - 4 * (NIT - 1);
    // bytes per point: 8 mod 16 dwords, free of bank conflicts (as k_conv's)
    static constexpr int PS = C == 16 ? 32 : 96;
    static constexpr int WB = NCH * NB * 256;                  // one conv's weights: [step][nb][lane group][i], 16 bytes
    static constexpr int W1 = NX * PS, W2 = W1 + WB, ZO = W2 + WB;      // ... a 16-byte zero
    static constexpr int B1 = ZO + 16, B2 = B1 + C * 4, HO = B2 + C * 4, DO = align16(HO + (NH * C + NH) * 4);
    static constexpr int TOTAL = DO + 2 * 64;
    static constexpr int SCH = C * 2 / 16, NQ = NX * SCH, NPF = (NQ + NTH - 1) / NTH;
    static constexpr int CPX = C * 2 / 16, NRC = TC * CPX / 64;
    static constexpr int OP = C == 32 ? 80 : C * 2;            // bytes per pixel of a staged row (64 would collide)
    static_assert(TOTAL <= 160 * 1024 && TR * TC * OP <= NX * PS && (TC * CPX) % 64 == 0, "LDS of the block kernel");
};

template <int C, int NH>
__global__ void __launch_bounds__(NTH, 2)
k_block(BlockArgs a, Geometry geo)
{
    using L = BL<C, NH>;
    constexpr bool HEAD = NH > 0;
    constexpr int NB = L::NB, NIT = L::NIT, PS = L::PS, SCH = L::SCH, NPF = L::NPF;
    extern __shared__ v4f smem[];
    char *sT = reinterpret_cast<char *>(smem);
    float *sB1 = reinterpret_cast<float *>(sT + L::B1), *sB2 = reinterpret_cast<float *>(sT + L::B2);
    float *sH = reinterpret_cast<float *>(sT + L::HO);
    int *sdec = reinterpret_cast<int *>(sT + L::DO);

    const ConvArgs &ca = a.c;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kq = lane >> 4;
    const int dd = ca.d, blk = ca.blk;

    // the weights, the last step's lane groups past the ninth tap left out
    for (int i = tid; i < NIT * NB * 64; i += NTH) {
        const int m = i / (NB * 64), r = i - m * (NB * 64), nb = r / 64, ln = r & 63;
        const bool full = m < NIT - 1;
        if (full || (ln >> 4) < L::REM) {
            const int o = (full ? i : (NIT - 1) * NB * 64 + nb * L::REM * 16 + ln) * 16;
            *reinterpret_cast<v4f *>(sT + L::W1 + o) = static_cast<const v4f *>(a.w1)[i];
            *reinterpret_cast<v4f *>(sT + L::W2 + o) = static_cast<const v4f *>(ca.wpk)[i];
        }
    }
    if (tid == 0) *reinterpret_cast<v4f *>(sT + L::ZO) = v4f{0.f, 0.f, 0.f, 0.f};
    for (int i = tid; i < C; i += NTH) {
        sB1[i] = a.b1[i];
        sB2[i] = ca.bias[i];
    }
    if constexpr (HEAD)
        for (int i = tid; i < NH * C + NH; i += NTH) sH[i] = ca.head[i];

    const int64_t T = geo.dyn ? ld_const(geo.dyn + DYN_TILES + blk) : geo.tiles[blk];
    const int nfr = geo.dyn ? (int)ld_const(geo.dyn + DYN_NF) : geo.nf;
    const int xcd = blockIdx.x % NXCD, slot = blockIdx.x / NXCD, nslot = gridDim.x / NXCD;
    const int64_t chunk = (T + NXCD - 1) / NXCD;
    const int64_t t0 = (int64_t)xcd * chunk, t1 = min(T, t0 + chunk);

    // loads of a tile's x, as k_conv's: off the frame they read zero
    v4f pf[NPF];
    // (Addresses are computed anew per tile, through `fresh`: kept, the many
    // lane-dependent ones of a tile would take the registers of the sums.)
    auto anew = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    auto fresh = [&](int v) { return C <= 32 ? v : anew(v); };
    auto issue = [&](const TileDec &r) {
        const int tid = fresh(threadIdx.x);
        const __amdgpu_buffer_rsrc_t rin =
            buf_rsrc(const_cast<char *>(static_cast<const char *>(ca.in)) + r.act * (C * 2), 0x7FFFFFFFu);
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const int q0 = tid + k * NTH, q = q0 < L::NQ ? q0 : L::NQ - 1;
            const int pt = q / SCH, ch = q - pt * SCH;
            const int ii = pt / XW - 2, jj = pt - (pt / XW) * XW - 2;
            const bool ok = q0 < L::NQ && (unsigned)(r.y0 + dd * ii) < (unsigned)r.h && (unsigned)(r.x0 + dd * jj) < (unsigned)r.w;
            pf[k] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                                rin, ok ? (r.a0 + ii * r.rs + jj * r.cs) * (C * 2) + ch * 16 : BUF_OOB, 0, 0));
        }
    };
    // Byte offset from a lane's tap-0 point (rows of `pw` points) of K chunk
    // 4 m + kq: see k_conv.
    auto chunk_off = [&](int m, int pw, int kq) {
        constexpr int CH8 = L::CH8;
        auto tap_off = [pw](int t) { return ((t / 3) * pw + t % 3) * PS; };
        const int tb = 4 * m / CH8, r = 4 * m - tb * CH8, tn = tb + 1 < 9 ? tb + 1 : 4;
        return kq * 16 + (kq >= CH8 - r ? tap_off(tn) + (r - CH8) * 16 : tap_off(tb) + r * 16);
    };
    auto weights = [&](int m, const char *w, v4f (&av)[NB]) {      // w: the lane's first fragment
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if (m == NIT - 1 && L::REM < 4) {
                const char *q = w + (m * NB * 64 + nb * L::REM * 16) * 16;
                av[nb] = *reinterpret_cast<const v4f *>(kq < L::REM ? q : sT + L::ZO);
            } else {
                av[nb] = *reinterpret_cast<const v4f *>(w + (m * NB + nb) * 1024);
            }
        }
    };
    auto mm = [](const v4f &w, const v4f &x, v4f &d) {
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, w), __builtin_bit_cast(v8bf, x), d, 0, 0, 0);
    };
    TileWalk walk;
    TileDec n{};
    int64_t ti = t0 + slot;
    if (ti < t1) {
        n = walk.tile(ca, geo, nfr, TR, TC, ti);
        issue(n);
        if (wave == 0) publish_tile(sdec, lane, walk.tile(ca, geo, nfr, TR, TC, ti + nslot < t1 ? ti + nslot : ti));
    }
#pragma unroll
    for (int k = 0; k < NPF; ++k) asm volatile("" : : "v"(pf[k]));
    for (int par = 0; ti < t1; ti += nslot, par ^= 1) {
        const int Y0 = n.y0, X0 = n.x0, H = n.h, W = n.w, A0 = n.a0, RS = n.rs, CS = n.cs;
        const int64_t px_off = n.px, act = n.act;
        __syncthreads();   // the previous tile's LDS reads are done (and weights staged)
        const int ts = fresh(tid);
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const int q = ts + k * NTH;
            if (q < L::NQ) {
                const int pt = q / SCH, ch = q - pt * SCH;
                *reinterpret_cast<v4f *>(sT + pt * PS + ch * 16) = pf[k];
            }
        }
        __syncthreads();
        n = pickup_tile(sdec + 16 * par);      // the next tile, or this one again past the last
        issue(n);
        __builtin_amdgcn_sched_barrier(0);     // (loads stay ahead of the MFMAs they overlap)

        // t: N blocks of this wave
        auto conv1 = [&](auto cnt) {
            constexpr int N = decltype(cnt)::value;
            // this lane's points of t: point 16 (wave + 8 i) + j of the 10 x 66 (past
            // the last: computed as point 0, and not kept)
            const int p0 = fresh(16 * wave + j);
            const char *w1 = sT + anew(L::W1 + lane * 16);
            v4f acc[N][NB];
            int base[N], mrow[N], mcol[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int p = p0 + 128 * i;
                mrow[i] = p < NM ? p / MW : 0;
                mcol[i] = p < NM ? p - (p / MW) * MW : 0;
                base[i] = (mrow[i] * XW + mcol[i]) * PS;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[i][nb] = v4f{0.f, 0.f, 0.f, 0.f};
            }
            // (the operands of step m + 1 are read while the MFMAs of step m run)
            v4f av[2][NB], bv[2][N];
            auto operands = [&](int m) {
                const int co = chunk_off(m, XW, fresh(kq));
                weights(m, w1, av[m & 1]);
#pragma unroll
                for (int i = 0; i < N; ++i) bv[m & 1][i] = *reinterpret_cast<const v4f *>(sT + base[i] + co);
            };
            operands(0);
#pragma unroll
            for (int m = 0; m < NIT; ++m) {
                if (m + 1 < NIT) operands(m + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int i = 0; i < N; ++i) mm(av[m & 1][nb], bv[m & 1][i], acc[i][nb]);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();                   // every wave has read x: t goes over it
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const bool in = (unsigned)(Y0 + dd * (mrow[i] - 1)) < (unsigned)H && (unsigned)(X0 + dd * (mcol[i] - 1)) < (unsigned)W;
                const bool keep = p0 + 128 * i < NM;
                char *t = sT + (mrow[i] * MW + mcol[i]) * PS + kq * 8;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const v4f v = relu4(acc[i][nb] + *reinterpret_cast<const v4f *>(sB1 + nb * 16 + kq * 4));
                    const uint2 pk{bf16_pack2(v[0], v[1]), bf16_pack2(v[2], v[3])};
                    if (keep) *reinterpret_cast<uint2 *>(t + nb * 32) = in ? pk : uint2{0u, 0u};
                }
            }
        };
        if (LO < HI && wave < NBLK - 8 * LO) conv1(std::integral_constant<int, HI>{});
        else conv1(std::integral_constant<int, LO>{});

        // the residual (x at this wave's row) while conv2 runs
        const int yo = Y0 + dd * wave;
        const bool row_ok = yo < H;
        const int Ar = A0 + wave * RS;
        v4u rc[HEAD ? 1 : L::NRC];
        uint2 rr[HEAD ? NB : 1][HEAD ? PB : 1];
        const int ln = fresh(lane);
        const __amdgpu_buffer_rsrc_t rres =
            buf_rsrc(const_cast<char *>(static_cast<const char *>(ca.in)) + act * (C * 2), 0x7FFFFFFFu);
        if constexpr (!HEAD) {
#pragma unroll
            for (int i = 0; i < L::NRC; ++i) {
                const int q = ln + 64 * i, px = q / L::CPX, part = q - px * L::CPX;
                rc[i] = __builtin_amdgcn_raw_buffer_load_b128(
                    rres, row_ok && X0 + dd * px < W ? (Ar + px * CS) * (C * 2) + part * 16 : BUF_OOB, 0, 0);
            }
        } else {
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const int c = 16 * p + j;
                const int o = row_ok && X0 + dd * c < W ? (Ar + c * CS) * (C * 2) + kq * 8 : BUF_OOB;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    rr[nb][p] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rres, o + nb * 32, 0, 0));
            }
        }
        if (wave == 0 && ti + nslot < t1) {
            const int64_t t2 = ti + 2 * nslot;
            publish_tile(sdec + 16 * (par ^ 1), lane, walk.tile(ca, geo, nfr, TR, TC, t2 < t1 ? t2 : ti + nslot));
        }
        __syncthreads();                       // t is complete
        v4f acc[PB][NB];
#pragma unroll
        for (int p = 0; p < PB; ++p)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[p][nb] = v4f{0.f, 0.f, 0.f, 0.f};
        v4f av[2][NB], bv[2][PB];
        const char *w2 = sT + anew(L::W2 + lane * 16);
        auto operands = [&](int m) {
            const char *xb = sT + (wave * MW + j) * PS + chunk_off(m, MW, fresh(kq));
            weights(m, w2, av[m & 1]);
#pragma unroll
            for (int p = 0; p < PB; ++p) bv[m & 1][p] = *reinterpret_cast<const v4f *>(xb + 16 * p * PS);
        };
        operands(0);
#pragma unroll
        for (int m = 0; m < NIT; ++m) {
            if (m + 1 < NIT) operands(m + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int p = 0; p < PB; ++p) mm(av[m & 1][nb], bv[m & 1][p], acc[p][nb]);
            __builtin_amdgcn_sched_barrier(0);
        }

        // epilogue, as k_conv's: the row passes through LDS (over t) so that it
        // moves in whole 16-byte lanes, or feeds the head
        const int osh = ca.out_shift, om = (1 << osh) - 1;
        const int ohd = (H + om) >> osh, owd = (W + om) >> osh;
        const int osub = (yo & om) << osh, oiy = yo >> osh;
        auto out_point = [&](int xo) { return ((osub + (xo & om)) * ohd + oiy) * owd + (xo >> osh); };
        char *sO = sT + wave * (TC * L::OP);
        if constexpr (!HEAD) {
            __syncthreads();                   // every wave has read t
#pragma unroll
            for (int i = 0; i < L::NRC; ++i) {
                const int q = ln + 64 * i, px = q / L::CPX;
                *reinterpret_cast<v4u *>(sO + px * L::OP + (q - px * L::CPX) * 16) = rc[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
        auto value = [&](int p, int nb, const uint2 &u) {     // what is stored, as BF16 pairs
            v4f v = acc[p][nb] + *reinterpret_cast<const v4f *>(sB2 + nb * 16 + kq * 4);
            v += v4f{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                     __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u)};
            v = relu4(v);
            return uint2{bf16_pack2(v[0], v[1]), bf16_pack2(v[2], v[3])};
        };
        if constexpr (HEAD) {
            constexpr int N = head_blocks<NH, C>(PB);
#pragma unroll
            for (int p0 = 0; p0 < PB; p0 += N) {
                float hh[N][NH] = {};
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    v4f vp[N];
#pragma unroll
                    for (int p = 0; p < N; ++p) {
                        const uint2 pk = value(p0 + p, nb, rr[nb][p0 + p]);
                        vp[p] = v4f{__uint_as_float(pk.x << 16), __uint_as_float(pk.x & 0xFFFF0000u),
                                    __uint_as_float(pk.y << 16), __uint_as_float(pk.y & 0xFFFF0000u)};
                    }
                    head_add<NH, C>(hh, sH, nb * 16 + kq * 4, vp);
                }
#pragma unroll
                for (int p = 0; p < N; ++p) {
                    const int xo = X0 + dd * (16 * (p0 + p) + j);
                    head_store(hh[p], sH + NH * C, ca.maps + NH * px_off + (int64_t)yo * W + xo, (int64_t)H * W, kq, xo < W && row_ok);
                }
            }
        } else {
#pragma unroll
            for (int p = 0; p < PB; ++p)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    uint2 *so = reinterpret_cast<uint2 *>(sO + (16 * p + j) * L::OP + (nb * 16 + kq * 4) * 2);
                    *so = value(p, nb, *so);
                }
        }
        if constexpr (!HEAD) {
            const __amdgpu_buffer_rsrc_t orow = buf_rsrc(static_cast<char *>(ca.out) + act * (C * 2), 0x7FFFFFFFu);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            const int le = fresh(lane);
#pragma unroll
            for (int i = 0; i < L::NRC; ++i) {
                const int q = le + 64 * i, px = q / L::CPX, part = q - px * L::CPX, xo = X0 + dd * px;
                const v4u d = *reinterpret_cast<const v4u *>(sO + px * L::OP + part * 16);
                __builtin_amdgcn_raw_buffer_store_b128(d, orow, row_ok && xo < W ? out_point(xo) * (C * 2) + part * 16 : BUF_OOB, 0, 0);
            }
        }
    }
}

template <int C, int NH>
hipError_t launch(const BlockArgs &a, const Geometry &g, int ncu, hipStream_t s)
{
    auto kern = k_block<C, NH>;
    constexpr int bytes = BL<C, NH>::TOTAL;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
        attr = true;
    }
    int per = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, NTH, bytes) != hipSuccess || per < 1) per = 1;
    int grid = (int)std::min<int64_t>(g.tiles[a.c.blk], (int64_t)per * ncu);
    grid = std::max(NXCD, grid / NXCD * NXCD);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NTH), bytes, s, a, g);
    return hipGetLastError();
}

template <int C>
hipError_t launch_c(const BlockArgs &a, const Geometry &g, int ncu, hipStream_t s)
{
    if (!a.c.head) return launch<C, 0>(a, g, ncu, s);
    return a.c.nh == 10 ? launch<C, 10>(a, g, ncu, s) : launch<C, 5>(a, g, ncu, s);
}

}  // namespace

// Up to 32 channels always (net A, 4 x 2048^2: the two layers of a block 1164 us,
// the block 904; passes, two layers | block, us: 64^2 68 | 54, 600^2 160 | 131, 901 x
// 1400 357 | 294; 16 channels 64^2 53 | 42, 600^2 108 | 93, 901 x 1400 193 | 185).  At
// 48 channels the second weights leave no room for a second workgroup's overlap and
// a full chip is slower this way (net B, 4 x 2048^2: 1733 us against 1941); while the
// tiles are at most two rounds of one workgroup per CU, one launch less counts for
// more (passes: 4 x 128^2 187 | 172, 500^2, 512 tiles, 273 | 246; 600^2, 750 to 1280,
// 365 | 368; 700^2 439 | 460).
bool block_takes(int C, int precision, int tr, int64_t tiles, int ncu)
{
    return precision == DL_BF16 && tr == TR && (C <= 32 || (C == 48 && tiles <= 2 * (int64_t)ncu));
}

hipError_t launch_block(int C, const BlockArgs &a, const Geometry &g, int ncu, hipStream_t s)
{
    switch (C) {
    case 16: return launch_c<16>(a, g, ncu, s);
    case 32: return launch_c<32>(a, g, ncu, s);
    case 48: return launch_c<48>(a, g, ncu, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dloc
