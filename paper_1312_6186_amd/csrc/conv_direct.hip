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

// Times in us, fits over 3 x 3 and 5 x 5 layers of 8 to 384 channels on 3 to 480 pixels square, 1500 to 400000 pixels (fp32: 90 %
// of the times within 15 %; bf16: 80 % within 25 %; the general engine within 10 and 15 %).
struct DirectRates {
    double launch, load, store;   // the launch; a patch load per thread ahead of the loop; the epilogue of an MFMA block
    double mma, filters;          // a K step: per MFMA block of a wave, and per block of columns what its filters take from L1 at least
    double large;                 // what a block takes in a wave tile of eight and more, which reads less per MFMA
    double pos1, pos3;            // a window position at least, with the filters one and three positions ahead
    double apart, single;         // what several workgroups on a CU do not hide of one's time; slowdown of chunks of one K step
};
constexpr DirectRates kRatesF32 = {4.7, 0.16, 0.5, 0.215, 0, 1, 0, 0, 0.06, 1.2}, kRatesBf16 = {3.3, 0, 1.0, 0.0113, 0.0195, 0.85, 0.155, 0.083, 0.6, 1.8};
constexpr double kPatchUs = 35e-6;   // a byte of patch: 28 GB/s for each CU while all of them fetch

double direct_us(int es, int ks, int nchunks, const Tile &t, const Gather &a, int N, int groups)
{
    const DirectRates &q = es == 2 ? kRatesBf16 : kRatesF32;
    const Fit f = fit(es, ks, nchunks, t, a);
    const int npos = a.kh * a.kw, blocks = t.mb * t.nb, registers = blocks > 8 ? 1 : blocks >= 3 ? 2 : 4;   // workgroups of four waves per CU
    const int per_cu = std::max(1, std::min((int)(163840 / f.lds), registers));
    const double position = ks * t.nb * std::max(q.mma * t.mb * (blocks >= 8 ? q.large : 1.0), q.filters) * (ks == 1 ? q.single : 1.0);
    const double least = es == 2 && blocks <= 4 && ks >= 2 && npos % 3 == 0 ? q.pos3 : q.pos1;
    const double alone = (double)nchunks * npos * std::max(position, least) + q.load * f.npl + q.store * blocks;
    const long M = (long)a.N * a.H * a.W, tiles = ((M + 32 * t.mb * t.wm - 1) / (32 * t.mb * t.wm)) * ((N + 32 * t.nb * t.wn - 1) / (32 * t.nb * t.wn)) * groups;
    return q.launch + rounds_us(tiles, per_cu, [&](int r) {
        return std::max(alone, r * nchunks * (npos * position + kPatchUs * f.patch_bytes) + q.apart * alone);
    });
}
// The general engine: tiles of 128 x 128 (half empty for up to 64 columns), K tiles of 128 bytes.
double engine_us(int es, const Gather &a, int N)
{
    const long M = (long)a.N * a.H * a.W, tiles = ((M + 127) / 128) * ((N + 127) / 128), kt = ((long)a.kh * a.kw * a.C * es + 127) / 128;
    const double half = N > 64 ? 1.0 : es == 2 ? 0.73 : 0.55;
    return es == 2 ? 1.9 + rounds_us(tiles, 2, [&](int r) { return 4.5 + half * kt * (r == 1 ? 0.54 : 0.94); })
                   : 1.2 + rounds_us(tiles, 2, [&](int r) { return 5.2 + half * kt * (r == 1 ? 2.06 : 3.98); });
}

}  // namespace

// The groups of a grouped layer count as column tiles of one launch; the general engine has a launch for each.  200 layers of 2 to 8 groups (8 to 192 channels a
// group, 3 x 3 and 5 x 5, 5 to 200 pixels wide, 1 to 256 images, both types), passes with one such layer: 1.002 times the better of the two on average, two more
// than 1.05 times (fp32 24 -> 40 5 x 5 on 17 x 88, 134 images, 1290 us, engine 1132); against a launch of conv_direct a group 0.82 (median of 150), at most 1.02.
DirectPlan plan_direct(int dtype, const Gather &a, int N, int groups)
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
    // In bf16 chunks of one K step are too short to hide a chunk's barrier and its filters: with several of them the general engine
    // is the faster one (80 -> 192 channels 5 x 5 on 8 x 8, 2591 images 187 us there, 280 here; over 176 such layers the best tile
    // shape took 0.7 to 2.2 times the engine's time, 1.1 on average).
    if (es == 2 && d.ks == 1 && d.nchunks > 1) return DirectPlan();
    const long M = (long)a.N * a.H * a.W;
    double best_cost = 0, cost_us = 0, best_us = 0;
    int by_cost = -1, by_time = -1;
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
        const long tiles = ((M + 32 * t.mb * t.wm - 1) / (32 * t.mb * t.wm)) * ((N + 32 * t.nb * t.wn - 1) / (32 * t.nb * t.wn)) * groups;
        const double cost = (double)((tiles + 255) / 256) * (t.mb * t.nb) * (t.wm * t.wn / 4.0) / eff, us = direct_us(es, d.ks, d.nchunks, t, a, N, groups);
        if (by_cost < 0 || cost < best_cost) { by_cost = v; best_cost = cost; cost_us = us; }
        if (by_time < 0 || us < best_us) { by_time = v; best_us = us; }
    }
    // That shape is measured inside steps, but knows neither the patch nor how many workgroups share a CU: where another one's
    // modelled time is a tenth shorter, that one (192 -> 96 channels 3 x 3 on 32 x 32, 272 images: 144 us in 192 x 128, one
    // workgroup to a CU, 117 in 128 x 128, two).  And the general engine keeps the layers for which its modelled time is the shortest:
    // a patch has kh - 1 more image rows than its tile, so on wide images it is many times as large, costs the workgroups that
    // would share the CU and is late (us, engine / here: fp32 48 -> 32 channels 3 x 3 on 128 x 192, 5 images 69 / 165; bf16
    // 96 -> 16 on 32 x 255, 26 images 47 / 110, 64 -> 128 on 64 x 480, 6 images 44 / 102).
    const int tile = cost_us > 1.1 * best_us ? by_time : by_cost;
    if (tile < 0 || groups * engine_us(es, a, N) < (tile == by_time ? best_us : cost_us)) return DirectPlan();
    d.tile = tile;
    d.npl = fit(es, d.ks, d.nchunks, kTiles[tile], a).npl;
    d.nblk_elems = (size_t)d.nchunks * npos * d.ks * 512;
    d.pack_elems = (size_t)((N + 31) / 32) * d.nblk_elems;
    if (d.pack_elems * groups * es > kMaxOperandBytes) return DirectPlan();
    return d;
}

// Few columns over few pixels: the general engine in K splits, where it is modelled a quarter faster.
bool split_is_faster(int dtype, const Gather &a, int N, int groups, const DirectPlan &d, size_t partials)
{
    double us = 0;
    return d.ks && plan_conv((long)a.N * a.H * a.W, N, (long)a.kh * a.kw * a.C, dtype, 1, partials, &us).splits > 1 &&
           groups * us < 0.75 * direct_us((int)dtype_size(dtype), d.ks, d.nchunks, kTiles[d.tile], a, N, groups);
}

int conv_direct(int dtype, const Gather &a, const void *wpack, int N, int groups, const Epilogue &ep, const DirectPlan &d, hipStream_t s)
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
    p.w = Operand{wpack, (unsigned)(d.pack_elems * groups * es)};
    p.groups = groups; p.xg_bytes = (unsigned)(a.C * es); p.wg_bytes = (unsigned)(d.pack_elems * es);
    p.nblk_bytes = (unsigned)(d.nblk_elems * es); p.nblks = (N + 31) / 32;
    p.tiles_n = (N + 32 * t.nb * t.wn - 1) / (32 * t.nb * t.wn);
    p.dW = make_fastdiv((uint32_t)a.W); p.dHW = make_fastdiv((uint32_t)(a.H * a.W));
    const long grid = (long)((p.M + 32 * t.mb * t.wm - 1) / (32 * t.mb * t.wm)) * p.tiles_n * groups;
    if (grid <= 0 || grid > 0x7fffffffL) return -1;
    const auto launch = dtype == kBF16 ? (ep.mask_src ? launch_direct_bf16_bwd : launch_direct_bf16_fwd) : (ep.mask_src ? launch_direct_f32_bwd : launch_direct_f32_fwd);
    return launch(d.tile, d.ks, p, ep, (unsigned)grid, f.lds, s);
}

}  // namespace asgd
