// Filter gradient of stride-1 convolutions over equal grids in 16-bit data:
// dW[co][(ky, kx, ci)] = sum over pixels m of dY[m][co] * X[m + (ky - pad) W + (kx - pad)][ci].
//
// A workgroup of four waves owns 32 MB WM output channels and, for one window row ky, ALL window columns kx of 32 WN input
// channels, over a range of pixels (split-K).  With channel-last storage the inputs of the kx of one pixel are
// neighbouring pixels, so a tile of 64 pixels needs 64 dY lines and one run of 64 + KW - 1 X lines in LDS:
// a window column is the same read one line further, an immediate offset.  Lines whose pixel has no row ky inside the image
// are stored as zeros; a lane whose pixel has no column kx inside the image reads zeros kept behind the tiles.
// Both operands have the reduction index outermost and are transposed by the LDS read (ds_read_b64_tr_b16: a half wave
// takes 64 bytes of four lines, which have to lie in different banks: X lines are 64 or 192 bytes apart, the 64-byte
// groups of a dY line are XOR-ed with bits of the line).
//
// What bounds it: at one wave per SIMD, the instructions beside the MFMAs (a wave has issue slots for eight per MFMA), then
// the MFMAs.  Hence a wave owns the same 32 input channels for every kx (one address, no per-block arithmetic), and the
// fragments of K step s + 1, the LDS stores of the next tile and the fetches of the tile three ahead stand
// between the MFMAs one by one; the barrier of a tile stands a third into its last K step, whose fragments are in
// registers by then.  (With the moves bunched at the front of a K step and the barrier before it: 20 % slower.)
//
// us alone, before (128 x 128 tiles of the general engine, both operands in LDS, every window position gathered) -> after,
// 128 images, 5 x 5 on 27 x 27: 96 -> 256 channels 127 -> 110, in two groups of 48 -> 128 82 -> 74; 3 x 3 on 13 x 13:
// 256 -> 384 51 -> 46, 384 -> 384 71 -> 60, 384 -> 256 50 -> 46 (with 4 x 3 blocks and one
// workgroup per CU 53), in two groups 58 -> 38 (384) and 46 -> 32 (256).  Beside the
// data gradients on the other stream they also leave more of the LDS and L2 to those: a step with 128 images 1403 -> 1332.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "asgd_internal.h"
#include "mfma_common.h"

namespace asgd {

struct WgradArgs {
    Operand x, dy; unsigned pix, ldyb;     // bytes from one pixel to the next
    int HW, W, C, npix, co, N;             // C, co: channels of a group; npix: pixels of the tensor; N = KW * KW * C
    int chunks, tiles_m, sets, groups;
    int nkt, per;                          // tiles of 64 pixels, and tiles per split
    FastDiv dW, dHW;
    float *ws;                             // [split][group][co][N]
};

constexpr int kWgKT = 64;   // pixels per tile
typedef __attribute__((address_space(3))) short4v lds_short4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
// MFMA blocks of a wave up to which two workgroups share a CU (the registers of a wave are halved)
constexpr int kWgShared = 6;

template <int MB, int KW, int WM, int WN>
__global__ __launch_bounds__(256, MB * KW <= kWgShared ? 2 : 1) void conv_wgrad_kernel(WgradArgs p)
{
    static_assert(WM * WN == 4 && WN <= 2 && KW % 2 == 1, "four waves, 32 or 64 input channels");
    constexpr int KT = kWgKT, PAD = KW / 2, COT = 32 * MB * WM, DP = COT * 2;   // bytes of a dY line
    constexpr int SPL = DP / 16, PD = KT * SPL / 256;                    // 16-byte pieces per dY line, and per thread and tile
    constexpr int XS = 4 * WN, XP = WN == 1 ? 64 : 192;                  // pieces per X line, and bytes from one to the next
    constexpr int XL = KT + KW - 1, PX = (XL * XS + 255) / 256;          // X lines; pieces per thread and tile
    constexpr int DB = KT * DP, XB = XL * XP;
    constexpr int ZERO = 2 * DB + 2 * XB, ZB = (XL * XP + 255) / 256 * 256 + 256;
    constexpr int NMFMA = MB * KW, NITEM = MB + KW, NMOVE = PD + PX, LAST = KT / 16 - 1, BAR = NMFMA / 3;
    static_assert(XB + 16 <= ZB, "a piece past the run lands among the zeros in either stage");
    // a line of 256 bytes (mod 256) needs all four groups exchanged, one of 128 (mod 256) the two groups of a pair
    constexpr bool SW4 = DP % 256 == 0;
    __shared__ __attribute__((aligned(256))) uint4 smem4[(ZERO + ZB) / 16];
    const unsigned sm = (unsigned)(size_t)(const __attribute__((address_space(3))) uint4 *)smem4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b4 = lane >> 4, i16 = lane & 15, lrow = lane & 31, half = lane >> 5;
    int bid;
    {   // each XCD gets a contiguous range of workgroups: neighbours share their pixels
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = blockIdx.x & 7;
        bid = x * q + (x < r ? x : r) + (blockIdx.x >> 3);
    }
    const int set = bid % p.sets; bid /= p.sets;
    const int tm = bid % p.tiles_m; bid /= p.tiles_m;
    const int grp = bid % p.groups, split = bid / p.groups;
    const int ky = set / p.chunks, ci0 = (set - ky * p.chunks) * (32 * WN);
    const int kt0 = split * p.per, nt = min(p.nkt, kt0 + p.per) - kt0;   // >= 1
    const int wm = (wave % WM) * MB, wn = wave / WM;                     // in blocks of 32

    // ---- operands on their way to LDS: piece tid + 256 j of a tile
    const __amdgpu_buffer_rsrc_t drs = p.dy.rsrc(), xrs = p.x.rsrc();
    const int yshift = (ky - PAD) * p.W;
    unsigned dvo[PD], xcol[PX], xst[PX];
    static_for<0, PD>([&](auto j) ASGD_INLINE {
        const int s = tid + j * 256, line = s / SPL, ps = s - line * SPL;
        const int grp64 = (ps >> 2) ^ (SW4 ? (line & 3) : ((line >> 1) & 1));
        const int col = tm * COT + grp64 * 32 + (ps & 3) * 8;
        dvo[j] = col < p.co ? (unsigned)line * p.ldyb + (unsigned)(grp * p.co + col) * 2u : kInv;   // lines past the tensor lie past its bytes
    });
    static_for<0, PX>([&](auto j) ASGD_INLINE {
        const int s = tid + j * 256, line = s / XS, col = (s % XS) * 8;
        xcol[j] = (ci0 + col < p.C && line < XL) ? (unsigned)(grp * p.C + ci0 + col) * 2u : kInv;
        xst[j] = sm + (line < XL ? 2 * DB + (unsigned)(line * XP + col * 2) : (unsigned)ZERO);   // pieces past the run: more zeros
    });
    uint4 r[2][NMOVE];
    auto fetch = [&](auto setc, auto j, int m0) ASGD_INLINE {
        if constexpr (j < PD) {
            r[setc][j] = buf_ld16(drs, dvo[j] + (unsigned)m0 * p.ldyb);
        } else {
            // the pixel has a row ky iff shifting it by whole rows stays inside its image
            const int q = m0 - PAD + (tid + (j - PD) * 256) / XS, rem = q - (int)fdiv((uint32_t)q, p.dHW) * p.HW;
            unsigned off = (unsigned)(q + yshift) * p.pix + xcol[j - PD];
            asm volatile("" : "+v"(off));   // a select, not a branch around the product
            const bool ok = ((unsigned)q < (unsigned)p.npix) & ((unsigned)(rem + yshift) < (unsigned)p.HW) & (xcol[j - PD] != kInv);
            r[setc][j] = buf_ld16(xrs, ok ? off : kInv);
        }
    };
    auto put = [&](auto setc, auto j, auto stage) ASGD_INLINE {
        const uint4 v = r[setc][j];
        if constexpr (j < PD) *reinterpret_cast<lds_u32x4 *>(sm + (unsigned)tid * 16u + (stage * DB + j * 4096)) = u32x4{v.x, v.y, v.z, v.w};
        else *reinterpret_cast<lds_u32x4 *>(xst[j - PD] + stage * XB) = u32x4{v.x, v.y, v.z, v.w};
    };

    // ---- fragments: this lane supplies line 8 (b4 / 2) + i16 / 4 (+ 4) of a K step, four channels of it
    const int l0 = 8 * (b4 >> 1) + (i16 >> 2);
    unsigned aoff[MB];
    int ox[2 * (LAST + 1)];                // column of the lane's pixels
    static_for<0, MB>([&](auto mb) ASGD_INLINE {
        const int sw = SW4 ? (l0 & 3) : ((l0 >> 1) & 1);
        aoff[mb] = sm + (unsigned)(l0 * DP + (((wm + mb) ^ sw) << 6) + 32 * (b4 & 1) + 8 * (i16 & 3));
    });
    const unsigned xl = (unsigned)(l0 * XP + wn * 64 + 32 * (b4 & 1) + 8 * (i16 & 3));
    const unsigned xoff[2] = {sm + 2 * DB + xl, sm + 2 * DB + XB + xl}, zoff = sm + ZERO + (xl & 255u);
    static_for<0, 2 * (LAST + 1)>([&](auto h) ASGD_INLINE {
        const int m = kt0 * KT + (h / 2) * 16 + (h % 2) * 4 + l0;
        ox[h] = m - (int)fdiv((uint32_t)m, p.dW) * p.W;
    });
    const int adv = KT % p.W;
    auto tr = [&](unsigned a, unsigned b) ASGD_INLINE -> uint4 {
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_short4 *>(a));
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_short4 *>(b));
        const uint2 x = __builtin_bit_cast(uint2, lo), y = __builtin_bit_cast(uint2, hi);
        return make_uint4(x.x, x.y, y.x, y.y);
    };
    Frag<bf16_t> fa[2][MB], fb[2][KW];
    // fragment i of K step ks, in the order of first use: window column 0, the output channels, the other window columns
    auto item = [&](auto i, auto ks, auto stage) ASGD_INLINE {
        constexpr int SET = ks & 1;
        if constexpr (i == 0 || i > MB) {
            constexpr int kx = i == 0 ? 0 : i - MB, o = ks * 16 * XP + kx * XP;
            auto side = [&](int x) ASGD_INLINE -> unsigned {
                if constexpr (kx < PAD) return x >= PAD - kx ? xoff[stage] : zoff;
                else if constexpr (kx > PAD) return x < p.W - (kx - PAD) ? xoff[stage] : zoff;
                else return xoff[stage];
            };
            fb[SET][kx].v = tr(side(ox[2 * ks]) + o, side(ox[2 * ks + 1]) + (o + 4 * XP));
        } else {
            constexpr int o = stage * DB + ks * 16 * DP;
            fa[SET][i - 1].v = tr(aoff[i - 1] + o, aoff[i - 1] + (o + 4 * DP));
        }
    };

    f32x16 acc[KW][MB];
    static_for<0, KW>([&](auto i) ASGD_INLINE { static_for<0, MB>([&](auto j) ASGD_INLINE { acc[i][j] = f32x16{}; }); });
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    int m0 = kt0 * KT;
    static_for<0, NMOVE>([&](auto j) ASGD_INLINE { fetch(I0{}, j, m0); });
    static_for<0, NMOVE>([&](auto j) ASGD_INLINE { fetch(I1{}, j, m0 + KT); });
    for (int z = tid; z < ZB / 16; z += 256) *reinterpret_cast<lds_u32x4 *>(sm + ZERO + (unsigned)z * 16u) = u32x4{0u, 0u, 0u, 0u};
    static_for<0, NMOVE>([&](auto j) ASGD_INLINE { put(I0{}, j, I0{}); });
    static_for<0, NMOVE>([&](auto j) ASGD_INLINE { fetch(I0{}, j, m0 + 2 * KT); });
    m0 += 3 * KT;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    static_for<0, NITEM>([&](auto i) ASGD_INLINE { item(i, I0{}, I0{}); });

    // One tile out of LDS stage ST.  Register set 1 - ST holds the next tile; it is stored, and refilled with the tile three
    // ahead.  (Past the end of the range these are tiles that nobody multiplies.)
    auto tile = [&](auto st) ASGD_INLINE {
        constexpr int ST = decltype(st)::value, NX = 1 - ST;
        static_for<0, LAST + 1>([&](auto ks) ASGD_INLINE {
            constexpr int KS = decltype(ks)::value;
            static_for<0, NMFMA>([&](auto i) ASGD_INLINE {
                constexpr int I = decltype(i)::value;
                if constexpr (KS < LAST) {   // the next K step's fragments, spread over the MFMAs
                    static_for<0, NITEM>([&](auto j) ASGD_INLINE {
                        if constexpr (decltype(j)::value * NMFMA / NITEM == I) item(j, std::integral_constant<int, KS + 1>{}, st);
                    });
                } else {
                    if constexpr (I == BAR) {
                        // every wave has its last fragments of this stage, and has stored its part of the next one
                        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                        static_for<0, 2 * (LAST + 1)>([&](auto h) ASGD_INLINE { ox[h] += adv; ox[h] -= ox[h] >= p.W ? p.W : 0; });
                    }
                    static_for<0, NITEM>([&](auto j) ASGD_INLINE {
                        if constexpr (BAR + decltype(j)::value * (NMFMA - BAR) / NITEM == I) item(j, I0{}, std::integral_constant<int, NX>{});
                    });
                }
                static_for<0, (NMOVE + NMFMA - 1) / NMFMA>([&](auto k) ASGD_INLINE {
                    constexpr int J = I + NMFMA * decltype(k)::value;
                    if constexpr (J < NMOVE && KS == 1) put(std::integral_constant<int, NX>{}, std::integral_constant<int, J>{}, std::integral_constant<int, NX>{});
                    if constexpr (J < NMOVE && KS == 2) fetch(std::integral_constant<int, NX>{}, std::integral_constant<int, J>{}, m0);
                });
                mma(acc[I / MB][I % MB], fb[KS & 1][I / MB], fa[KS & 1][I % MB]);
                __builtin_amdgcn_sched_barrier(0x6);   // plain vector and scalar arithmetic may cross, nothing else
            });
        });
        m0 += KT;
    };
    for (int t = nt >> 1; t > 0; --t) {
        tile(I0{});
        tile(I1{});
    }
    if (nt & 1) tile(I0{});

    // acc[kx][mb][v]: channel (wm + mb) 32 + lrow, input channel wn 32 + 8 (v / 4) + 4 half + v % 4
    float *o = p.ws + (size_t)(split * p.groups + grp) * (size_t)p.co * (size_t)p.N;
    static_for<0, KW>([&](auto kx) ASGD_INLINE {
        static_for<0, 4>([&](auto g) ASGD_INLINE {
            const int ci = ci0 + wn * 32 + 8 * g + 4 * half, n = (ky * KW + kx) * p.C + ci;
            static_for<0, MB>([&](auto mb) ASGD_INLINE {
                const int m = tm * COT + (wm + mb) * 32 + lrow;
                if (ci < p.C && m < p.co)
                    *reinterpret_cast<f32x4 *>(o + (size_t)m * p.N + n) = f32x4{acc[kx][mb][4 * g], acc[kx][mb][4 * g + 1], acc[kx][mb][4 * g + 2], acc[kx][mb][4 * g + 3]};
            });
        });
    });
}

namespace {
struct WgTile { int mb, kw, wm, wn; };
constexpr WgTile kWgTiles[] = {{3, 3, 2, 2}, {2, 3, 2, 2}, {2, 5, 4, 1}, {2, 5, 2, 2}};
constexpr int kWgTileCount = 4;
}

// Partial sums are written and read again at the rate of a copy.
constexpr double kPartialUs = 0.37e-6 * 4;   // us per float

// M: output channels of a group; x: one group's input as a gather
//
// The tile shape and the number of pixel ranges (splits) with the smallest modelled time: the MFMA blocks of the busiest CU plus
// the partial sums.  Few pixels want few splits, and a small result many: with the chip filled whatever that cost, 256 -> 384
// channels on 13 x 13 at 4 images took 33 us in 11 splits (39 MB of partial sums; 17 in 2 splits of the narrower tile), 64 -> 128
// on 56 x 56 at 16 images 34 us in 157 (27 in 66), 64 -> 128 on 13 x 13 at 32 images 26 in 85.  The general engine (128 x 128
// tiles, both operands gathered for every window position) keeps the layers for which its modelled time is the smaller one (15,
// 29 and 15 us of these three), and those whose channels would be more than two fifths padding here: it skips waves that hold
// nothing but padding.  The times of a block and of a K tile are fits over 3 x 3 and 5 x 5 layers of 32 to 512 channels on 7 to
// 224 pixels square, 1 to 256 images (90 % of the times within 10 %, the general engine's within 20 %).
WgradPlan plan_wgrad(int dtype, int M, int groups, const Gather &x, size_t max_ws_floats)
{
    WgradPlan best;
    const size_t pixb = x.pix ? x.pix : (size_t)x.C * 2;
    if (dtype != kBF16 || x.sm != 1 || x.ds != 1 || x.Ho != x.H || x.Wo != x.W || x.kh != x.kw || 2 * x.pad != x.kw - 1 ||
        (x.rowb != 0 && x.rowb != (size_t)x.W * pixb) || pixb % 16 != 0 || x.C % 8 != 0 || M % 8 != 0)
        return best;
    const long npix = (long)x.N * x.H * x.W, nkt = (npix + kWgKT - 1) / kWgKT;
    const double result = (double)groups * M * x.kh * x.kw * x.C;
    double best_us = 0;
    for (int v = 0; v < kWgTileCount; ++v) {
        const WgTile &t = kWgTiles[v];
        if (t.kw != x.kw) continue;
        const int blocks = t.mb * t.kw;
        const bool shared = blocks <= kWgShared;                 // two workgroups of this shape fit a CU
        const long tiles = (long)groups * ((M + 32 * t.mb * t.wm - 1) / (32 * t.mb * t.wm)) * ((x.C + 32 * t.wn - 1) / (32 * t.wn)) * x.kh;
        const double useful = (double)groups * M * x.C * x.kh / ((double)tiles * (32.0 * t.mb * t.wm) * (32.0 * t.wn));
        if (useful < 0.6) continue;
        const long most = std::max(1L, std::min(nkt, (shared ? 512 : 256) / tiles));
        for (long splits = 1, per = nkt; splits <= most && splits * result <= (double)max_ws_floats;) {
            const double us = rounds_us(tiles * splits, shared ? 2 : 1, [&](int r) { return (!shared ? 0.085 : r == 1 ? 0.11 : 0.18) * blocks * per; }) + kPartialUs * splits * result;
            if (best.tile < 0 || us < best_us) { best.tile = v; best.splits = (int)splits; best_us = us; }
            if (per == 1) break;
            splits = (nkt + per - 2) / (per - 1);                // the fewest with fewer tiles each, none of them empty
            per = (nkt + splits - 1) / splits;
        }
    }
    if (best.tile < 0) return best;
    const long N = (long)x.kh * x.kw * x.C;
    const GemmPlan g = plan_gemm(M, N, npix, dtype, 128);        // what the general engine would run, once per group
    const long per = (nkt + g.splits - 1) / g.splits;
    const double general = groups * (rounds_us(((M + 127) / 128) * ((N + 127) / 128) * g.splits, 2, [&](int r) { return (r == 1 ? 0.34 : 0.87) * per; }) + kPartialUs * g.ws_floats);
    // a launch more per group there, one for the partial sums here; results that are stored where they belong from a whole sum
    // are scattered there
    if (general + 9.0 * (groups - 1) + (g.splits == 1 ? 1.0 : -1.0) < best_us) return WgradPlan();
    best.ws_floats = (size_t)best.splits * groups * M * N;
    return best;
}

int conv_wgrad(const void *dy, long ldy, int M, int groups, const Gather &x, const Epilogue &ep, const WgradPlan &plan, float *ws, Reduction *later, hipStream_t s)
{
    if (plan.tile < 0 || plan.tile >= kWgTileCount || kWgTiles[plan.tile].kw != x.kw || ep.mode != 1 || !ep.out_f32 || !ws || ((uintptr_t)ws & 15) || ((uintptr_t)dy & 15) || ((uintptr_t)x.x & 15) || ldy % 8) return -1;
    const WgTile &t = kWgTiles[plan.tile];
    WgradArgs p;
    const long npix = (long)x.N * x.H * x.W;
    const size_t dyb = ((size_t)(npix - 1) * ldy + (size_t)groups * M) * 2;
    if (dyb > kMaxOperandBytes || x.bytes > kMaxOperandBytes) return -1;
    p.x = Operand{x.x, (unsigned)x.bytes}; p.dy = Operand{dy, (unsigned)dyb};
    p.pix = x.pix ? (unsigned)x.pix : (unsigned)(x.C * 2); p.ldyb = (unsigned)(ldy * 2);
    p.HW = x.H * x.W; p.W = x.W; p.C = x.C; p.npix = (int)npix; p.co = M; p.N = x.kh * x.kw * x.C;
    p.chunks = (x.C + 32 * t.wn - 1) / (32 * t.wn); p.sets = p.chunks * x.kh;
    p.tiles_m = (M + 32 * t.mb * t.wm - 1) / (32 * t.mb * t.wm); p.groups = groups;
    p.nkt = (int)((npix + kWgKT - 1) / kWgKT); p.per = (p.nkt + plan.splits - 1) / plan.splits;
    p.dW = make_fastdiv((uint32_t)x.W); p.dHW = make_fastdiv((uint32_t)(x.H * x.W));
    p.ws = ws;
    const long grid = (long)p.sets * p.tiles_m * groups * plan.splits;
    if (grid <= 0 || grid > 0x7fffffffL || (long)(plan.splits - 1) * p.per >= p.nkt) return -1;
    const dim3 g((unsigned)grid), b(256);
    switch (plan.tile) {
    case 0: hipLaunchKernelGGL((conv_wgrad_kernel<3, 3, 2, 2>), g, b, 0, s, p); break;
    case 1: hipLaunchKernelGGL((conv_wgrad_kernel<2, 3, 2, 2>), g, b, 0, s, p); break;
    case 2: hipLaunchKernelGGL((conv_wgrad_kernel<2, 5, 4, 1>), g, b, 0, s, p); break;
    default: hipLaunchKernelGGL((conv_wgrad_kernel<2, 5, 2, 2>), g, b, 0, s, p); break;
    }
    return splitk_reduce(kBF16, ws, plan.splits, ep, groups * M, p.N, later, s);
}

}  // namespace asgd
