// Host side of conv_direct_kernel: where it applies, with which chunk and tile shape, and its launch.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "conv_direct.h"

namespace asgd {

namespace {

struct Tile { int mb, nb, wm, wn; };
#define ASGD_TILE_ROW(V, MB, NB, WM, WN) {MB, NB, WM, WN},
constexpr Tile kTiles[kDirectTiles] = {ASGD_DIRECT_TILES(ASGD_TILE_ROW)};
#undef ASGD_TILE_ROW

struct Fit { int npl; unsigned patch_bytes, lds; bool ok; };

// LDS layout of a tile shape, and whether it can run at all
Fit fit(int es, int ks, int nchunks, const Tile &t, const Gather &a)
{
    const int pieces = ks * es, sh = pieces > 4 ? 3 : pieces > 2 ? 2 : 1, pitch = ks * 16 * es + 16;
    const int nt = 64 * t.wm * t.wn, ppl = nt >> sh, pixels = 32 * t.mb * t.wm + (a.kh - 1) * a.W + a.kw - 1;
    Fit f;
    f.npl = (pixels + ppl - 1) / ppl;
    const long patch = ((long)f.npl * ppl * pitch + 255) / 256 * 256;
    const long lds = std::max(patch * (nchunks > 1 ? 2 : 1) + kDirectZero + nt * 16, (long)t.wm * t.wn * t.nb * 4096 + 32L * t.nb * t.wn * 4);
    f.ok = lds <= 163840 && (nchunks == 1 || f.npl <= direct_pieces(ks, a.kh * a.kw));
    f.patch_bytes = (unsigned)patch; f.lds = (unsigned)lds;
    return f;
}

}  // namespace

DirectPlan plan_direct(int dtype, const Gather &a, int N)
{
    DirectPlan d;
    const int es = (int)dtype_size(dtype), npos = a.kh * a.kw;
    const size_t pixb = a.pix ? a.pix : (size_t)a.C * es;
    if (!(a.sm == 1 && a.ds == 1 && a.Ho == a.H && a.Wo == a.W && npos > 1 && npos <= 32 && 2 * a.pad == a.kh - 1 && 2 * a.pad == a.kw - 1 &&
          (a.rowb == 0 || a.rowb == (size_t)a.W * pixb) && pixb % 16 == 0 && a.C % 8 == 0 && N % 8 == 0 && a.bytes <= kMaxOperandBytes))
        return d;
    // Channels per chunk: the K steps (of 16 channels) that pad the channel count least; among equals 64, then 32, then 48.
    const int order[4] = {4, 2, 3, 1};
    long best_steps = 0;
    for (int q = 0; q < 4; ++q) {
        const int ks = order[q];
        if (ks * es > 8) continue;
        const long steps = (long)((a.C + 16 * ks - 1) / (16 * ks)) * ks;
        if (d.ks == 0 || steps < best_steps) { d.ks = ks; best_steps = steps; }
    }
    d.nchunks = (a.C + 16 * d.ks - 1) / (16 * d.ks);
    const long M = (long)a.N * a.H * a.W;
    double best = 0;
    int tile = -1;
    for (int v = 0; v < kDirectTiles; ++v) {
        const Tile &t = kTiles[v];
        if (!direct_has(es, v, d.ks) || !fit(es, d.ks, d.nchunks, t, a).ok) continue;
        // Rounds of workgroups over the 256 CUs, times the MFMA blocks of a round, over the share of the matrix rate that the
        // shape reaches in its loop (measured in bf16 over the 3 x 3 and 5 x 5 layers at 32 to 256 images: larger wave tiles
        // read less per MFMA, so 0.61 for 96 x 96 down to 0.3 for 32 x 32; what counts most is how the tiles divide among
        // the CUs: 384 -> 256 channels at 128 images take 41 us in 170 tiles of 256 x 128 and 36 in 226 of 192 x 128, at
        // 77 images 38 and 26 in 204 of 128 x 128).  fp32 MFMAs take eight times as long: every shape keeps them busy.
        const double eff_bf16 = t.mb * t.nb >= 6 ? 0.61 : t.mb * t.nb >= 4 ? 0.57 : t.mb * t.nb == 3 ? 0.45 : t.mb == 2 ? 0.47 : t.nb == 2 ? 0.37 : 0.3;
        const double eff = es == 2 ? eff_bf16 : 0.8;
        const long tiles = ((M + 32 * t.mb * t.wm - 1) / (32 * t.mb * t.wm)) * ((N + 32 * t.nb * t.wn - 1) / (32 * t.nb * t.wn));
        const double cost = (double)((tiles + 255) / 256) * (t.mb * t.nb) * (t.wm * t.wn / 4.0) / eff;
        if (tile < 0 || cost < best) { tile = v; best = cost; }
    }
    if (tile < 0) { d.ks = 0; return d; }
    d.tile = tile;
    d.npl = fit(es, d.ks, d.nchunks, kTiles[tile], a).npl;
    d.nblk_elems = (size_t)d.nchunks * npos * d.ks * 512;
    d.pack_elems = (size_t)((N + 31) / 32) * d.nblk_elems;
    if (d.pack_elems * es > kMaxOperandBytes) { d.ks = 0; return d; }
    return d;
}

int conv_direct(int dtype, const Gather &a, const void *wpack, int N, const Epilogue &ep, const DirectPlan &d, hipStream_t s)
{
    const int es = (int)dtype_size(dtype);
    if (d.ks == 0 || ((uintptr_t)a.x & 15) || ((uintptr_t)wpack & 15) || ((uintptr_t)ep.out & 15) || (ep.ld & 7) || ep.mode || ep.drop || ep.out_f32) return -1;
    const Tile &t = kTiles[d.tile];
    const Fit f = fit(es, d.ks, d.nchunks, t, a);
    if (!f.ok) return -1;
    DirectConv p;
    p.x = Operand{a.x, (unsigned)a.bytes};
    p.pix = a.pix ? (unsigned)a.pix : (unsigned)(a.C * es);
    p.H = a.H; p.W = a.W; p.C = a.C; p.kh = a.kh; p.kw = a.kw; p.pad = a.pad; p.npos = a.kh * a.kw;
    p.M = a.N * a.H * a.W; p.N = N;
    p.nchunks = d.nchunks; p.npl = f.npl;
    p.patch_bytes = f.patch_bytes; p.patch_off2 = d.nchunks > 1 ? f.patch_bytes : 0;
    p.w = Operand{wpack, (unsigned)(d.pack_elems * es)};
    p.nblk_bytes = (unsigned)(d.nblk_elems * es); p.nblks = (N + 31) / 32;
    p.tiles_n = (N + 32 * t.nb * t.wn - 1) / (32 * t.nb * t.wn);
    p.dW = make_fastdiv((uint32_t)a.W); p.dHW = make_fastdiv((uint32_t)(a.H * a.W));
    const long grid = (long)((p.M + 32 * t.mb * t.wm - 1) / (32 * t.mb * t.wm)) * p.tiles_n;
    if (grid <= 0 || grid > 0x7fffffffL) return -1;
    const auto launch = dtype == kBF16 ? (ep.mask_src ? launch_direct_bf16_bwd : launch_direct_bf16_fwd) : (ep.mask_src ? launch_direct_f32_bwd : launch_direct_f32_fwd);
    return launch(d.tile, d.ks, p, ep, (unsigned)grid, f.lds, s);
}

}  // namespace asgd
