// MFMA GEMM engine for gfx950: one kernel template serves the convolutions
// (forward, data gradient, filter gradient, all as implicit GEMMs) and the fully
// connected layers.  C[M][N] = sum_k A[m][k] * B[n][k], fp32 accumulation.
//
// Geometry (identical in bytes for both element types): a workgroup owns a
// 128 x 128 tile of C; one K tile is 128 bytes per row (64 bf16 or 32 fp32).
// Two workgroups share a CU.  The GEMMs run 8 wave64 per workgroup (wave tile
// 64 x 32, four waves per SIMD), except the fp32 convolution filter gradient,
// which runs 4 (wave tile 64 x 64).  Operands arrive through range-checked 16-byte
// buffer loads (out-of-range pieces read as zeros), two K tiles ahead, into
// registers, and go from there to one of two LDS stages, so that one barrier per
// K tile suffices.  An operand whose memory has K contiguous sits in LDS as rows
// x 8 slots of 16 bytes, the slot index XOR-swizzled with the row so that
// fragment reads and stores are spread over the banks.  An operand whose memory
// has the GEMM row contiguous and K strided (both operands of the filter
// gradients, the weights in the FC data gradient) is copied to LDS in that
// orientation and transposed by the LDS read itself (ds_read_b64_tr_b16).  The
// MFMA is issued with the B-matrix fragment as its first operand so that a lane
// ends up with four consecutive n for one m.  The output goes through LDS once
// more, so that a lane owns 8 consecutive columns of a row and a wave stores
// whole row segments as 16-byte vectors.  Workgroup ids are remapped so that each
// of the 8 XCDs (which receive ids round-robin) works on a contiguous range of
// tiles and its L2 sees neighbouring tiles' shared operand rows.  A wave runs at
// raised priority while it multiplies a tile, and a wave whose part of the tile
// lies outside C does not multiply at all.
//
// Stride-1 convolutions whose output grid equals their input grid run
// conv_direct_kernel (conv_direct.h) instead.  Small fully-connected products run
// lone_kernel, weight gradients over a minibatch outer_kernel (both below); few
// output channels or columns take narrower tiles of the same engine (Cfg32, Cfg64,
// CfgN32).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "asgd_internal.h"
#include "mfma_common.h"
#include "reduce.h"

namespace asgd {

// Tile configuration: block tile BM x BN, WAVES_M x WAVES_N wave64s, DEPTH K tiles in flight in registers,
// MINB workgroups per CU the register budget is sized for.
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, int DEPTH_, int MINB_> struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, DEPTH = DEPTH_, MINB = MINB_;
    static constexpr int NT = 64 * WAVES_M_ * WAVES_N_;
    static constexpr int MB = BM_ / WAVES_M_ / 32, NB = BN_ / WAVES_N_ / 32;   // MFMA 32x32 blocks per wave
    static_assert((BM_ / WAVES_M_) % 32 == 0 && (BN_ / WAVES_N_) % 32 == 0, "wave tiles in blocks of 32");
};
using Cfg128 = TileCfg<128, 128, 2, 2, 2, 2>;   // 256 threads (wave tile 64x64), two workgroups per CU: two waves per SIMD
using Cfg128w8 = TileCfg<128, 128, 2, 4, 2, 2>; // 512 threads (wave tile 64x32), two workgroups per CU: four waves per SIMD

// filter gradients of few output channels: in fp32 three workgroups a CU of 32 rows, otherwise two
template <typename T> using Cfg32 = TileCfg<32, 128, 1, 4, 2, sizeof(T) == 4 ? 6 : 4>;
using Cfg64 = TileCfg<64, 128, 2, 2, 2, 4>;
using CfgN32 = TileCfg<128, 32, 4, 1, 2, 4>;    // convolutions of up to 32 output columns: 256 threads (wave tile 32x32), four workgroups per CU

FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f;
    f.d = d;
    uint32_t sh = 0;
    while ((1ull << sh) < d) ++sh;
    f.sh = sh;
    f.mul = (uint32_t)((((1ull << 32) * ((1ull << sh) - d)) / d) + 1);
    if (d == 1) { f.mul = 0; f.sh = 0; }
    return f;
}

// ------------------------------------------------------------------ loaders
// value of lane S of the caller's quad (4 consecutive lanes)
template <int S> __device__ __forceinline__ unsigned quad_bcast(unsigned v)
{
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, S * 0x55, 0xF, 0xF, true);
}

// Direct loaders hand out 16-byte pieces of a row that are contiguous in K.
template <typename T> struct PlainK {
    static constexpr bool kTrans = false;
    Operand op; unsigned ldb; int rows, K;   // ldb: bytes from one row to the next
    struct Row { unsigned off; };
    struct KPos { int k; unsigned koff; };
    __device__ __forceinline__ Row row(int r) const { return Row{r < rows ? (unsigned)r * ldb : kInv}; }
    __device__ __forceinline__ KPos kpos(int k) const { return KPos{k, k < K ? (unsigned)k * (unsigned)sizeof(T) : kInv}; }
    __device__ __forceinline__ void advance(KPos &kp, int dk) const
    {
        kp.k += dk;
        kp.koff = kp.k < K ? (unsigned)kp.k * (unsigned)sizeof(T) : kInv;
    }
    __device__ __forceinline__ unsigned voff(const Row &r, const KPos &kp) const { return r.off + kp.koff; }
};

// Implicit-GEMM gather, unit divisor (forward convolution, stride-1 data gradient).
// All per-row work is done once: a row keeps the byte offset of its window origin
// and a bit mask saying which window positions (ky, kx) fall inside the image; a K
// position keeps the byte offset of (ky, kx, c) relative to a window origin and
// the bit of its window position.  Fetching a piece is then one mask test, one add
// and one select.  WIDE = windows of more than 32 positions (two 16-bit masks, one per axis).
template <typename T, bool WIDE> struct GatherK {
    static constexpr bool kTrans = false;
    Operand op;
    unsigned rowb, pix;  // bytes from one image row / one pixel to the next
    int H, W, C, Ho, Wo, kh, kw, sm, pad, M;
    int adv_px, adv_c;   // one K tile = adv_px whole pixels + adv_c channels
    FastDiv dWo, dHoWo, dC, dkw;
    struct Row { unsigned off, mask; };
    struct KPos { int ky, kx, c; unsigned delta, bit; };
    __device__ __forceinline__ Row row(int m) const
    {
        if (m >= M) return Row{0u, 0u};
        const int n = (int)fdiv((uint32_t)m, dHoWo);
        const int rem = m - n * (Ho * Wo);
        const int oy = (int)fdiv((uint32_t)rem, dWo);
        const int ox = rem - oy * Wo;
        const int y0 = oy * sm - pad, x0 = ox * sm - pad;
        // ky is inside for max(0,-y0) <= ky < min(kh, H-y0); the same along x
        const int ylo = max(0, -y0), yhi = max(ylo, min(kh, H - y0));
        const int xlo = max(0, -x0), xhi = max(xlo, min(kw, W - x0));
        const unsigned ym = ((1u << yhi) - 1u) & ~((1u << ylo) - 1u), xm = ((1u << xhi) - 1u) & ~((1u << xlo) - 1u);
        unsigned mask = 0;
        if (WIDE) {
            mask = ym | (xm << 16);
        } else {
            for (int a = 0; a < kh; ++a)
                if ((ym >> a) & 1u) mask |= xm << (a * kw);
        }
        return Row{(unsigned)(n * H + y0) * rowb + (unsigned)x0 * pix, mask};
    }
    __device__ __forceinline__ unsigned bit_of(int ky, int kx) const
    {
        const unsigned b = WIDE ? ((1u << (ky & 15)) | (1u << (16 + kx))) : (1u << ((ky * kw + kx) & 31));
        return ky < kh ? b : 0u;
    }
    __device__ __forceinline__ KPos kpos(int k) const
    {
        const int t = (int)fdiv((uint32_t)k, dC);
        const int ky = (int)fdiv((uint32_t)t, dkw);
        const int kx = t - ky * kw, c = k - t * C;
        return KPos{ky, kx, c, (unsigned)ky * rowb + (unsigned)kx * pix + (unsigned)c * (unsigned)sizeof(T), bit_of(ky, kx)};
    }
    // branch-free: no divergent control flow between the loads of a pipeline step
    __device__ __forceinline__ void advance(KPos &kp, int) const
    {
        kp.c += adv_c;
        const int wrap = kp.c >= C ? 1 : 0;
        kp.c -= wrap * C;
        kp.kx += adv_px + wrap;
        const int up = (int)fdiv((uint32_t)kp.kx, dkw);
        kp.kx -= up * kw;
        kp.ky += up;
        kp.delta = (unsigned)kp.ky * rowb + (unsigned)kp.kx * pix + (unsigned)kp.c * (unsigned)sizeof(T);
        kp.bit = bit_of(kp.ky, kp.kx);
    }
    __device__ __forceinline__ unsigned voff(const Row &r, const KPos &kp) const
    {
        const bool ok = WIDE ? (kp.bit != 0u && (r.mask & kp.bit) == kp.bit) : ((r.mask & kp.bit) != 0u);
        return ok ? r.off + kp.delta : kInv;
    }
};

// The same gather with a divisor (data gradient of a strided convolution): positions
// that are not multiples of the stride contribute nothing.  Rare, kept simple.
template <typename T> struct GatherKS {
    static constexpr bool kTrans = false;
    Operand op; unsigned pix;   // bytes from one pixel to the next
    int H, W, C, Ho, Wo, kh, kw, sm, ds, pad, M;
    FastDiv dWo, dHoWo, dC, dkw;
    struct Row { int pix0, y0, x0; };  // pix0 < 0: row out of range
    struct KPos { int ky, kx, c; };
    __device__ __forceinline__ Row row(int m) const
    {
        if (m >= M) return Row{-1, 0, 0};
        const int n = (int)fdiv((uint32_t)m, dHoWo);
        const int rem = m - n * (Ho * Wo);
        const int oy = (int)fdiv((uint32_t)rem, dWo);
        const int ox = rem - oy * Wo;
        return Row{n * H * W, oy * sm - pad, ox * sm - pad};
    }
    __device__ __forceinline__ KPos kpos(int k) const
    {
        const int t = (int)fdiv((uint32_t)k, dC);
        const int ky = (int)fdiv((uint32_t)t, dkw);
        return KPos{ky, t - ky * kw, k - t * C};
    }
    __device__ __forceinline__ void advance(KPos &kp, int dk) const
    {
        kp.c += dk;
        while (kp.c >= C) {
            kp.c -= C;
            if (++kp.kx == kw) { kp.kx = 0; ++kp.ky; }
        }
    }
    __device__ __forceinline__ unsigned voff(const Row &r, const KPos &kp) const
    {
        if (r.pix0 < 0 || kp.ky >= kh) return kInv;
        int y = r.y0 + kp.ky, xx = r.x0 + kp.kx;
        if (y < 0 || xx < 0) return kInv;
        if ((y % ds) != 0 || (xx % ds) != 0) return kInv;
        y /= ds; xx /= ds;
        if (y >= H || xx >= W) return kInv;
        return (unsigned)(r.pix0 + y * W + xx) * pix + (unsigned)kp.c * (unsigned)sizeof(T);
    }
};

// Row-contiguous loaders: memory has the GEMM row index contiguous and the
// reduction index strided ([k][rows]).  The tile is copied to LDS in that same
// orientation, 16 bytes (8 or 4 consecutive rows) at a time; the transposition
// the MFMA needs happens in the LDS read (ds_read_b64_tr_b16 for 16-bit data).
// A thread keeps one column of 16-byte pieces (Col) and walks down the K axis.
template <typename T> struct PlainT {
    static constexpr bool kTrans = true, kShared = false;
    Operand op; unsigned ldb; int rows, K;
    struct Col { unsigned off; };
    struct KState { int k; unsigned koff; };
    __device__ __forceinline__ Col col(int row0) const { return Col{row0 < rows ? (unsigned)row0 * (unsigned)sizeof(T) : kInv}; }
    __device__ __forceinline__ KState kstate(int k) const { return KState{k, k < K ? (unsigned)k * ldb : kInv}; }
    __device__ __forceinline__ void advance(KState &ks, int dk) const
    {
        ks.k += dk;
        ks.koff = ks.k < K ? ks.koff + (unsigned)dk * ldb : kInv;   // once past K it stays past K
    }
    __device__ __forceinline__ unsigned voff(const Col &c, const KState &ks) const { return c.off + ks.koff; }
};

// Filter-gradient gather: rows enumerate (ky, kx, c) (fixed per column of pieces), the reduction index
// enumerates output pixels m = (n, oy, ox).  What depends on the pixel alone (the byte offset of its window
// origin and the mask of window positions that fall inside the image) is computed once per pixel and K tile:
// the four lanes of a quad copy the same column for four different pixels, each works out one pixel and the
// quad exchanges the results with DPP moves.  A column keeps its offset inside the window and the mask bits of
// its (ky, kx); a piece is fetched iff the pixel's mask has both bits.
template <typename T> struct GatherT {
    static constexpr bool kTrans = true, kShared = true;
    Operand op;
    unsigned rowb, pix;  // bytes from one image row / one pixel to the next
    int H, W, C, Ho, Wo, kh, kw, sm, pad, M, Krows;
    FastDiv dWo, dHo, dHoWo, dC, dkw;
    struct Col { unsigned off, bits; };   // out-of-range columns: bits no pixel mask can have
    struct KState { int m, n, oy, ox; };
    struct Pixel { unsigned base, mask; };
    __device__ __forceinline__ Col col(int row0) const
    {
        if (row0 >= Krows) return Col{0u, 0xFFFFFFFFu};
        const int t = (int)fdiv((uint32_t)row0, dC);
        const int ky = (int)fdiv((uint32_t)t, dkw);
        const int kx = t - ky * kw, c = row0 - t * C;
        return Col{(unsigned)(ky - pad) * rowb + (unsigned)(kx - pad) * pix + (unsigned)c * (unsigned)sizeof(T),
                   (1u << ky) | (1u << (16 + kx))};
    }
    __device__ __forceinline__ KState kstate(int m) const
    {
        const int n = (int)fdiv((uint32_t)m, dHoWo);
        const int rem = m - n * (Ho * Wo);
        const int oy = (int)fdiv((uint32_t)rem, dWo);
        return KState{m, n, oy, rem - oy * Wo};
    }
    __device__ __forceinline__ void advance(KState &ks, int dk) const
    {
        ks.m += dk;
        ks.ox += dk;
        const int q = (int)fdiv((uint32_t)ks.ox, dWo);
        ks.ox -= q * Wo;
        ks.oy += q;
        const int q2 = (int)fdiv((uint32_t)ks.oy, dHo);
        ks.oy -= q2 * Ho;
        ks.n += q2;
    }
    __device__ __forceinline__ Pixel pixel(const KState &ks) const
    {
        const int y0 = ks.oy * sm - pad, x0 = ks.ox * sm - pad;
        const int ylo = max(0, -y0), yhi = max(ylo, min(kh, H - y0));
        const int xlo = max(0, -x0), xhi = max(xlo, min(kw, W - x0));
        const unsigned ym = ((1u << yhi) - 1u) & ~((1u << ylo) - 1u), xm = ((1u << xhi) - 1u) & ~((1u << xlo) - 1u);
        return Pixel{(unsigned)(ks.n * H + ks.oy * sm) * rowb + (unsigned)(ks.ox * sm) * pix, ks.m < M ? (ym | (xm << 16)) : 0u};
    }
    __device__ __forceinline__ unsigned voff(const Col &c, unsigned base, unsigned mask) const
    {
        return (mask & c.bits) == c.bits ? c.off + base : kInv;
    }
};

// ------------------------------------------------------------------ staging
template <typename T, class L, int ROWS, int NT, int DEPTH, bool kTrans = L::kTrans> struct Stage;

template <typename T, class L, int ROWS, int NT, int DEPTH> struct Stage<T, L, ROWS, NT, DEPTH, false> {
    static constexpr int SLOTS = ROWS * 8 / NT;
    typename L::Row rows[SLOTS];
    typename L::KPos kp;
    uint4 r[DEPTH][SLOTS];   // DEPTH K tiles in flight
    unsigned wo[2];      // LDS byte offset of slot 0 / slot 1; slot s sits s/2 * 64 rows further
    __device__ __forceinline__ void init(const L &l, int row0, int k0, int tid, int)
    {
        static_for<0, 2>([&](auto par) ASGD_INLINE {
            const int row = (tid >> 3) + par * (NT / 8);
            wo[par] = (unsigned)(row * 8 + ((tid & 7) ^ swz(row))) * 16u;
        });
        static_for<0, SLOTS>([&](auto s) ASGD_INLINE { rows[s] = l.row(row0 + (tid >> 3) + s * (NT / 8)); });
        kp = l.kpos(k0 + (tid & 7) * Geo<T>::CH);
    }
    // fetch the K tile at the cursor into register set RB and advance the cursor
    template <int RB> __device__ __forceinline__ void load(const L &l)
    {
        const __amdgpu_buffer_rsrc_t rs = l.op.rsrc();
        static_for<0, SLOTS>([&](auto s) ASGD_INLINE { r[RB][s] = buf_ld16(rs, l.voff(rows[s], kp)); });
        l.advance(kp, Geo<T>::BK);
    }
    template <int RB> __device__ __forceinline__ void store(uint4 *sm, int tid) const
    {
        // rows 64 apart share the swizzle, so the offset of slot s is that of slot s%2 plus a constant
        char *base = reinterpret_cast<char *>(sm);
        static_for<0, SLOTS>([&](auto s) ASGD_INLINE {
            *reinterpret_cast<uint4 *>(base + wo[s % 2] + (s / 2) * (2 * (NT / 8) * 128)) = r[RB][s];
        });
    }
};

template <typename T, class L, int ROWS, int NT, int DEPTH> struct Stage<T, L, ROWS, NT, DEPTH, true> {
    static constexpr int CPL = ROWS * (int)sizeof(T) / 16;   // 16-byte pieces per K line
    static constexpr int LPP = NT / CPL;                     // K lines covered by one pass of the workgroup
    static constexpr int SLOTS = Geo<T>::BK / LPP;
    static constexpr int NKS = L::kShared ? 1 : SLOTS;
    static_assert(NT % CPL == 0 && Geo<T>::BK % LPP == 0, "tile / thread-count mismatch");
    static_assert(!L::kShared || ((SLOTS == 4 || SLOTS == 2) && CPL % 4 == 0), "a quad shares one column and owns its K lines");
    typename L::Col c;
    typename L::KState ks[NKS];   // shared form: the K line of slot (tid & 3) only
    uint4 r[DEPTH][SLOTS];
    unsigned wo;   // LDS byte offset of slot 0
    __device__ __forceinline__ void init(const L &l, int row0, int k0, int tid, int)
    {
        const int cc = tid % CPL, line = tid / CPL;
        c = l.col(row0 + cc * (16 / (int)sizeof(T)));
        if constexpr (L::kShared) ks[0] = l.kstate(k0 + line + (tid & (SLOTS - 1)) * LPP);
        else static_for<0, SLOTS>([&](auto s) ASGD_INLINE { ks[s] = l.kstate(k0 + line + s * LPP); });
        wo = (unsigned)(line * TransTile<T, ROWS>::LINE + cc * 16);
    }
    template <int RB> __device__ __forceinline__ void load(const L &l)
    {
        const __amdgpu_buffer_rsrc_t rs = l.op.rsrc();
        if constexpr (L::kShared) {
            const auto px = l.pixel(ks[0]);
            l.advance(ks[0], Geo<T>::BK);
            static_for<0, SLOTS>([&](auto s) ASGD_INLINE {
                r[RB][s] = buf_ld16(rs, l.voff(c, quad_bcast<s>(px.base), quad_bcast<s>(px.mask)));
            });
        } else {
            static_for<0, SLOTS>([&](auto s) ASGD_INLINE {
                r[RB][s] = buf_ld16(rs, l.voff(c, ks[s]));
                l.advance(ks[s], Geo<T>::BK);
            });
        }
    }
    template <int RB> __device__ __forceinline__ void store(uint4 *sm, int) const
    {
        char *base = reinterpret_cast<char *>(sm);
        static_for<0, SLOTS>([&](auto s) ASGD_INLINE {
            *reinterpret_cast<uint4 *>(base + wo + s * (LPP * TransTile<T, ROWS>::LINE)) = r[RB][s];
        });
    }
};

// ------------------------------------------------------------------ kernel
// One K tile out of LDS.  The fragments of K step ks+1 are requested before the
// MFMAs of step ks are issued, so the LDS latency hides behind the matrix pipe.
template <typename T, int MB, int NB, class FOA, class FOB>
__device__ __forceinline__ void compute_tile(const uint4 *sA, const uint4 *sB, f32x16 (&acc)[NB][MB], const FOA &foA, const FOB &foB)
{
    constexpr int KS = Geo<T>::KSTEPS;
    const char *pa = reinterpret_cast<const char *>(sA), *pb = reinterpret_cast<const char *>(sB);
    Frag<T> fa[2][MB], fb[2][NB];
    static_for<0, MB>([&](auto mb) ASGD_INLINE { fa[0][mb].template read<0, mb>(pa, foA); });
    static_for<0, NB>([&](auto nb) ASGD_INLINE { fb[0][nb].template read<0, nb>(pb, foB); });
    static_for<0, KS>([&](auto ks) ASGD_INLINE {
        constexpr int cur = ks % 2, nxt = (ks + 1) % 2;
        if constexpr (ks + 1 < KS) {
            static_for<0, MB>([&](auto mb) ASGD_INLINE { fa[nxt][mb].template read<ks + 1, mb>(pa, foA); });
            static_for<0, NB>([&](auto nb) ASGD_INLINE { fb[nxt][nb].template read<ks + 1, nb>(pb, foB); });
        }
        static_for<0, NB>([&](auto nb) ASGD_INLINE { static_for<0, MB>([&](auto mb) ASGD_INLINE { mma(acc[nb][mb], fb[cur][nb], fa[cur][mb]); }); });
    });
}

// Output of a block tile: the accumulators go through LDS so that every lane ends up with 8 consecutive columns
// of one row and a wave stores whole row segments (the MFMA layout gives a lane 4 columns of one row and its
// neighbours other rows).  The whole tile is staged at once, BM rows of BN floats without padding: the 16-byte
// chunk index is XOR-ed with the row, so that the 16 lanes of a write (16 rows, one chunk column) and the 16
// lanes of a read (one row, 16 chunks) each touch every bank once.
// acc[nb][mb][v]: m = wm + mb*32 + lrow, n = wn + nb*32 + 8*(v/4) + 4*half + v%4
// Second half of the output phase: NTALL threads take the staged tile out of LDS, eight columns of a row each.
template <typename T, class Cfg, int NTALL>
__device__ __forceinline__ void emit_tile(const uint4 *smem, const Epilogue &ep, int tm, int tn, int split, int M, int N, float *ws,
                                          const float (&bias8)[8], int tid)
{
    constexpr int BM = Cfg::BM, BN = Cfg::BN;
    constexpr int CPR = BN / 4;                       // 16-byte chunks per row
    const float4 *stg = reinterpret_cast<const float4 *>(smem);
    constexpr int LPR = BN / 8, RPR = NTALL / LPR;   // lanes per row, rows per round
    static_for<0, BM / RPR>([&](auto r) ASGD_INLINE {
        const int row = r * RPR + tid / LPR, chunk = (tid % LPR) * 2;
        const int m = tm * BM + row, n0 = tn * BN + chunk * 4;
        if (m < M && n0 < N) {
            const float4 lo = stg[row * CPR + (chunk ^ (row & (CPR - 1)))];
            const float4 hi = stg[row * CPR + ((chunk + 1) ^ (row & (CPR - 1)))];
            float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            if (ws) store8<float>(ws + ((long)split * M + m) * N + n0, v);
            else epilogue8<T>(ep, m, n0, v, bias8);
        }
    });
}

// The push of a parameter gradient done in place of storing it (Epilogue::upd_w): the staged tile is the gradient of
// a BM x BN block of parameters.  A thread asks for the parameters and momenta of all its rows before the barrier
// that completes the staging, so that the whole block (2 x 64 KB) is in flight at once; the arithmetic is that of
// the streaming update kernel, contraction for contraction, and the worker copy is rounded as the snapshot rounds.
__device__ __forceinline__ uint32_t bf16_bits_rne(uint32_t u)
{
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (u >> 16) | 0x0040u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
// Four consecutive parameters at p with gradient g: w, mo their old values and momenta, acc what has been added up so far.
template <typename T> __device__ __forceinline__ void push4(const Epilogue &ep, long p, f32x4 g, f32x4 w, f32x4 mo, f32x4 acc)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float wo = w[e], vo = mo[e];
        const float t = __builtin_fmaf(ep.upd_wd, wo, g[e]);
        const float vn = __builtin_fmaf(ep.upd_mu, vo, -(ep.upd_lr * t));
        mo[e] = vn;
        w[e] = wo + vn;
    }
    __builtin_nontemporal_store(w, reinterpret_cast<f32x4 *>(__builtin_assume_aligned(ep.upd_w + p, 16)));
    __builtin_nontemporal_store(mo, reinterpret_cast<f32x4 *>(__builtin_assume_aligned(ep.upd_v + p, 16)));
    if (ep.out) __builtin_nontemporal_store(g, reinterpret_cast<f32x4 *>(__builtin_assume_aligned(static_cast<float *>(ep.out) + p, 16)));
    if (ep.upd_acc) __builtin_nontemporal_store(ep.upd_acc_first ? g : acc + g, reinterpret_cast<f32x4 *>(__builtin_assume_aligned(ep.upd_acc + p, 16)));
    if constexpr (sizeof(T) == 4) {
        for (int c = 0; c < ep.upd_copies; ++c) *reinterpret_cast<f32x4 *>(__builtin_assume_aligned(static_cast<float *>(ep.upd_copy[c]) + p, 16)) = w;
    } else {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        u32x2 o;
        o.x = bf16_bits_rne(__float_as_uint(w[0])) | (bf16_bits_rne(__float_as_uint(w[1])) << 16);
        o.y = bf16_bits_rne(__float_as_uint(w[2])) | (bf16_bits_rne(__float_as_uint(w[3])) << 16);
        for (int c = 0; c < ep.upd_copies; ++c) *reinterpret_cast<u32x2 *>(__builtin_assume_aligned(static_cast<bf16_t *>(ep.upd_copy[c]) + p, 8)) = o;
    }
}
template <typename T, class Cfg, int NTALL>
__device__ __forceinline__ void update_tile(const uint4 *smem, const Epilogue &ep, int tm, int tn, int M, int N, int tid)
{
    // a lane owns 4 consecutive columns, so that the 16-byte pieces of one store instruction are consecutive in
    // memory (32 lanes = 512 bytes of a row): whole lines leave the CU at once
    constexpr int BM = Cfg::BM, BN = Cfg::BN, CPR = BN / 4, RPR = NTALL / CPR, R = BM / RPR;
    const float4 *stg = reinterpret_cast<const float4 *>(smem);
    const int chunk = tid % CPR, n0 = tn * BN + chunk * 4;
    f32x4 w[R], mo[R], acc[R];
    const bool add = ep.upd_acc && !ep.upd_acc_first;
    static_for<0, R>([&](auto r) ASGD_INLINE {
        const int m = tm * BM + r * RPR + tid / CPR;
        if (m < M && n0 < N) {
            const long p = (long)m * ep.ld + n0;
            if (add) acc[r] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(__builtin_assume_aligned(ep.upd_acc + p, 16)));
            w[r] = *reinterpret_cast<const f32x4 *>(__builtin_assume_aligned(ep.upd_w + p, 16));
            mo[r] = *reinterpret_cast<const f32x4 *>(__builtin_assume_aligned(ep.upd_v + p, 16));
        }
    });
    __syncthreads();
    static_for<0, R>([&](auto r) ASGD_INLINE {
        const int row = r * RPR + tid / CPR, m = tm * BM + row;
        if (m < M && n0 < N) {
            const float4 g4 = stg[row * CPR + (chunk ^ (row & (CPR - 1)))];
            push4<T>(ep, (long)m * ep.ld + n0, f32x4{g4.x, g4.y, g4.z, g4.w}, w[r], mo[r], acc[r]);
        }
    });
}

// The output phase of the Cfg::NT threads that hold accumulators; NTALL >= Cfg::NT threads of the workgroup take part in
// its second half (the others pass the two barriers and call emit_tile themselves).
template <typename T, class Cfg, int SMEM_BYTES, int NTALL = Cfg::NT, bool PUSH = false>
__device__ __forceinline__ void output_tile(uint4 *smem, f32x16 (&acc)[Cfg::NB][Cfg::MB], const Epilogue &ep, int tm, int tn, int split, int M,
                                            int N, float *ws, const float (&bias8)[8], int tid, int wm, int wn)
{
    constexpr int BM = Cfg::BM, BN = Cfg::BN, MB = Cfg::MB, NB = Cfg::NB;
    constexpr int CPR = BN / 4;                   // 16-byte chunks per row
    static_assert(BM * BN * 4 <= SMEM_BYTES, "staging area");
    float4 *stg = reinterpret_cast<float4 *>(smem);
    const int lane = tid & 63, lrow = lane & 31, half = lane >> 5;
    __syncthreads();
    static_for<0, MB>([&](auto mb) ASGD_INLINE {
        const int row = wm + mb * 32 + lrow;
        static_for<0, NB>([&](auto nb) ASGD_INLINE {
            static_for<0, 4>([&](auto g) ASGD_INLINE {
                const int chunk = (wn + nb * 32 + 8 * g + 4 * half) / 4;
                stg[row * CPR + (chunk ^ (row & (CPR - 1)))] =
                    make_float4(acc[nb][mb][4 * g], acc[nb][mb][4 * g + 1], acc[nb][mb][4 * g + 2], acc[nb][mb][4 * g + 3]);
            });
        });
    });
    if constexpr (PUSH) {   // only the kernel instance that serves the fully-connected weight gradient carries this path
        static_assert(NTALL == Cfg::NT, "every thread of the workgroup takes part in the push");
        if (ep.upd_w) { update_tile<T, Cfg, NTALL>(smem, ep, tm, tn, M, N, tid); return; }
    }
    __syncthreads();
    emit_tile<T, Cfg, NTALL>(smem, ep, tm, tn, split, M, N, ws, bias8, tid);
}

// Software pipeline.  LDS holds two stages so that one barrier per K tile
// suffices; DEPTH K tiles are in flight in registers while another is being
// multiplied out of LDS.  At the top of step t, LDS stage t%2 holds tile t and
// the register sets hold tiles t+1 .. t+DEPTH-1 (possibly still arriving).
template <typename T, class Cfg, class LA, class LB>
__global__ __launch_bounds__(Cfg::NT, Cfg::MINB) void gemm_kernel(LA la, LB lb, Epilogue ep, int M, int N, int nkt, int kt_per_split,
                                                                int tiles_m, int tiles_n, float *ws)
{
    constexpr int BK = Geo<T>::BK, BM = Cfg::BM, BN = Cfg::BN, NT = Cfg::NT, MB = Cfg::MB, NB = Cfg::NB, DEPTH = Cfg::DEPTH;
    constexpr int TA = LA::kTrans ? TransTile<T, BM>::BYTES : BM * 128, TB = LB::kTrans ? TransTile<T, BN>::BYTES : BN * 128;
    __shared__ uint4 smem[2 * (TA + TB) / 16];   // two stages of A and B tiles; reused to stage the output
    uint4 (*sA)[TA / 16] = reinterpret_cast<uint4 (*)[TA / 16]>(smem);
    uint4 (*sB)[TB / 16] = reinterpret_cast<uint4 (*)[TB / 16]>(smem + 2 * TA / 16);
    const int tid = threadIdx.x;
    // XCD-aware remap: ids congruent mod 8 run on one XCD; give that XCD a contiguous range of tiles
    int bid;
    {
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = blockIdx.x & 7;
        bid = x * q + (x < r ? x : r) + (blockIdx.x >> 3);
    }
    const int tn = bid % tiles_n; bid /= tiles_n;
    const int tm = bid % tiles_m;
    const int split = bid / tiles_m;
    const int kt0 = split * kt_per_split;
    const int nt = min(nkt, kt0 + kt_per_split) - kt0;   // K tiles of this workgroup (>= 1)

    Stage<T, LA, BM, NT, DEPTH> stA;
    Stage<T, LB, BN, NT, DEPTH> stB;
    stA.init(la, tm * BM, kt0 * BK, tid, 0);
    stB.init(lb, tn * BN, kt0 * BK, tid, NT / 2);

    f32x16 acc[NB][MB];
    static_for<0, NB>([&](auto i) ASGD_INLINE { static_for<0, MB>([&](auto j) ASGD_INLINE { acc[i][j] = f32x16{}; }); });

    const int lane = tid & 63, wave = tid >> 6;
    const int wm = (wave % Cfg::WAVES_M) * (BM / Cfg::WAVES_M), wn = (wave / Cfg::WAVES_M) * (BN / Cfg::WAVES_N);
    FragOff<T, LA::kTrans, BM> foA;
    FragOff<T, LB::kTrans, BN> foB;
    foA.init(wm, lane);
    foB.init(wn, lane);
    // a wave whose whole tile lies outside C (96 output columns in a tile of 128: a quarter of the waves) only helps
    // to move the operands; wave-uniform
    const bool busy = __builtin_amdgcn_readfirstlane((tm * BM + wm < M && tn * BN + wn < N) ? 1 : 0) != 0;

    // register set that receives tile j is j % DEPTH (tile 0 goes through set 0 straight into LDS stage 0)
    stA.template load<0>(la); stB.template load<0>(lb);
    if constexpr (DEPTH == 2) { stA.template load<1>(la); stB.template load<1>(lb); }
    // every output row this thread writes has the same 8 columns: their bias is asked for behind the first tiles,
    // so that tile 0 does not wait for it (the parameters are cold in every cache, the tiles mostly are not)
    float bias8[8];
    load_bias8<T>(ep, tn * BN + (tid % (BN / 8)) * 8, bias8);
    stA.template store<0>(sA[0], tid); stB.template store<0>(sB[0], tid);
    // The loop body is two whole steps without a condition in it, so that the compiler knows exactly which fetches are
    // in flight at its head (with a conditional store it has to assume that those of two steps ago may be, and
    // waits for everything before it issues the next ones).  The store at the end of the last pair moves a tile that
    // exists only if the number of tiles is odd; otherwise it moves zeros that nobody reads.
    for (int i = nt >> 1; i > 0; --i) {
        // step t (even): multiply out of LDS stage 0, fetch tile t+DEPTH, then move tile t+1 into stage 1
        __syncthreads();
        stA.template load<0>(la); stB.template load<0>(lb);   // past the last tile this fetches zeros
        __builtin_amdgcn_s_setprio(1);   // the waves that multiply go first; those of the other workgroup are fetching or waiting
        if (busy) compute_tile<T, MB, NB>(sA[0], sB[0], acc, foA, foB);
        __builtin_amdgcn_s_setprio(0);
        stA.template store<DEPTH - 1>(sA[1], tid); stB.template store<DEPTH - 1>(sB[1], tid);
        // step t+1 (odd): multiply out of LDS stage 1, fetch tile t+1+DEPTH, then move tile t+2 into stage 0
        __syncthreads();
        stA.template load<DEPTH - 1>(la); stB.template load<DEPTH - 1>(lb);
        __builtin_amdgcn_s_setprio(1);
        if (busy) compute_tile<T, MB, NB>(sA[1], sB[1], acc, foA, foB);
        __builtin_amdgcn_s_setprio(0);
        stA.template store<0>(sA[0], tid); stB.template store<0>(sB[0], tid);
    }
    if (nt & 1) {
        __syncthreads();
        if (busy) compute_tile<T, MB, NB>(sA[0], sB[0], acc, foA, foB);
    }

    output_tile<T, Cfg, (int)sizeof(smem), Cfg::NT, LA::kTrans && LB::kTrans>(smem, acc, ep, tm, tn, split, M, N, ws, bias8, tid, wm, wn);
}

// Weight gradients of fully-connected layers, C[out][in] = sum over the minibatch: a short reduction, and C in fp32 is far more
// bytes than its operands, so what counts is that stores leave the CUs without a pause.  One LDS stage of K, an output
// phase in which every wave moves its own blocks through 4 KB of LDS without a barrier, and three workgroups a CU: the stores of one run under
// the loads of the others.  A wave's 32 columns of a row are one line of memory and leave in one instruction: non-temporal
// stores of whole lines.  (Plain stores straight from the accumulators, 32 bytes of a row at a time, take the same time
// alone, but the dirty lines they leave in L2 cost the data gradients beside them 4 % of a step.)
// 4096 x 9216 in bf16, 32 images: 54 -> 30 us (5.0 TB/s; a fill runs at 6.6), 77 images 47 -> 30; 4096 x 4096 24 -> 14; fp32, 128 images
// (two thirds of the matrix rate) 112 -> 105.
template <typename T>
__global__ __launch_bounds__(512, sizeof(T) == 2 ? 6 : 4) void outer_kernel(PlainT<T> la, PlainT<T> lb, float *out, long ld, int M, int N, int K, int tiles_n)
{
    constexpr int BK = Geo<T>::BK, KS = Geo<T>::KSTEPS, BYTES = TransTile<T, 128>::BYTES;
    __shared__ uint4 smem[2 * BYTES / 16];
    uint4 *sA = smem, *sB = smem + BYTES / 16;
    const int tid = threadIdx.x;
    int bid;
    {
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = blockIdx.x & 7;
        bid = x * q + (x < r ? x : r) + (blockIdx.x >> 3);
    }
    const int tm = bid / tiles_n, tn = bid - tm * tiles_n;
    Stage<T, PlainT<T>, 128, 512, 1> stA, stB;
    stA.init(la, tm * 128, 0, tid, 0);
    stB.init(lb, tn * 128, 0, tid, 0);
    f32x16 acc[2];
    acc[0] = f32x16{}; acc[1] = f32x16{};
    const int lane = tid & 63, wave = tid >> 6, wm = (wave & 1) * 64, wn = (wave >> 1) * 32;
    FragOff<T, true, 128> foA, foB;
    foA.init(wm, lane);
    foB.init(wn, lane);
    const bool busy = __builtin_amdgcn_readfirstlane((tm * 128 + wm < M && tn * 128 + wn < N) ? 1 : 0) != 0;
    stA.template load<0>(la); stB.template load<0>(lb);
    for (int k = 0; k < K; k += BK) {
        if (k) __syncthreads();
        stA.template store<0>(sA, tid); stB.template store<0>(sB, tid);
        __syncthreads();
        if (k + BK < K) { stA.template load<0>(la); stB.template load<0>(lb); }
        if (!busy) continue;
        static_for<0, KS>([&](auto ks) ASGD_INLINE {
            if (k + ks * 16 < K) {
                Frag<T> fa[2], fb;
                fb.template read<ks, 0>(reinterpret_cast<const char *>(sB), foB);
                static_for<0, 2>([&](auto i) ASGD_INLINE { fa[i].template read<ks, i>(reinterpret_cast<const char *>(sA), foA); });
                static_for<0, 2>([&](auto i) ASGD_INLINE { mma(acc[i], fb, fa[i]); });
            }
        });
    }
    // through LDS, each wave on its own: 32 columns of a row are one line of memory, a store instruction writes eight of them
    const int lrow = lane & 31, half = lane >> 5;
    __syncthreads();
    f32x4 *stg = reinterpret_cast<f32x4 *>(smem) + wave * 256;
    static_for<0, 2>([&](auto mb) ASGD_INLINE {
        static_for<0, 4>([&](auto g) ASGD_INLINE {
            stg[lrow * 8 + ((2 * g + half) ^ (lrow & 7))] = f32x4{acc[mb][4 * g], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]};
        });
        const int piece = lane & 7, n = tn * 128 + wn + piece * 4;
        static_for<0, 4>([&](auto r) ASGD_INLINE {
            const int row = r * 8 + (lane >> 3), m = tm * 128 + wm + mb * 32 + row;
            const f32x4 v = stg[row * 8 + (piece ^ (row & 7))];
            if (m < M && n < N) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(__builtin_assume_aligned(out + (long)m * ld + n, 16)));
        });
    });
}

// Products that a tile of 128 x 128 would put on a few CUs (the fully-connected layers of small nets): tiles of 16 x 16, whose K is
// dealt out to the waves of a workgroup in steps of 32, operands straight from L2 into registers one step ahead, the waves'
// sums added in LDS in their order.  What bounds it is the latency of a launch and of two or three trips to L2.  128 images, fp32,
// with the reduction of split sums / here: 576 -> 64 outputs forward 14.2 / 7.9 us, data gradient 12.1 / 4.1, weight gradient 15.2 / 4.4; 64 -> 10
// forward 10.0 / 4.4, gradients 9.1 and 7.8 / 4.5 and 4.2.
template <typename T> __device__ __forceinline__ void load_piece(Frag<T> &f, const PlainK<T> &l, __amdgpu_buffer_rsrc_t rs, unsigned off, int k)
{
    if constexpr (sizeof(T) == 2) {
        f.v = buf_ld16(rs, off + (k < l.K ? (unsigned)k * 2u : kInv));
    } else {
        f.v[0] = buf_ld16(rs, off + (k < l.K ? (unsigned)k * 4u : kInv));
        f.v[1] = buf_ld16(rs, off + (k + 4 < l.K ? (unsigned)(k + 4) * 4u : kInv));
    }
}
template <typename T> __device__ __forceinline__ void load_piece(Frag<T> &f, const PlainT<T> &l, __amdgpu_buffer_rsrc_t rs, unsigned off, int k)
{
    unsigned e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const unsigned o = off + (k + j < l.K ? (unsigned)(k + j) * l.ldb : kInv);
        if constexpr (sizeof(T) == 2) e[j] = (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)o, 0, 0);
        else e[j] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)o, 0, 0);
    }
    if constexpr (sizeof(T) == 2) {
        f.v = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
    } else {
        f.v[0] = make_uint4(e[0], e[1], e[2], e[3]);
        f.v[1] = make_uint4(e[4], e[5], e[6], e[7]);
    }
}
// eight K positions per lane, four groups of lanes: 32 of K
__device__ __forceinline__ void mma16(f32x4 &acc, const Frag<bf16_t> &first, const Frag<bf16_t> &second)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, first.v), __builtin_bit_cast(bf16x8, second.v), acc, 0, 0, 0);
}
__device__ __forceinline__ void mma16(f32x4 &acc, const Frag<float> &first, const Frag<float> &second)
{
    const uint32_t a[8] = {first.v[0].x, first.v[0].y, first.v[0].z, first.v[0].w, first.v[1].x, first.v[1].y, first.v[1].z, first.v[1].w};
    const uint32_t b[8] = {second.v[0].x, second.v[0].y, second.v[0].z, second.v[0].w, second.v[1].x, second.v[1].y, second.v[1].z, second.v[1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), acc, 0, 0, 0);
}
template <typename T> __device__ __forceinline__ unsigned row_offset(const PlainK<T> &l, int r) { return l.row(r).off; }
template <typename T> __device__ __forceinline__ unsigned row_offset(const PlainT<T> &l, int r) { return l.col(r).off; }
constexpr int kLoneWaves = 8;
template <typename T> struct LonePair {
    PlainT<T> wa, wb; Epilogue w_ep; int w_m, w_n, w_k, w_tiles_n, w_blocks;   // weight gradient: output gradients and inputs, K = images
    PlainK<T> da; PlainT<T> db; Epilogue d_ep; int d_m, d_n, d_k, d_tiles_n;   // data gradient: output gradients and weights, K = outputs
};
struct LoneShared { f32x4 part[kLoneWaves][64]; float sums[16][20]; };
// softmax cross-entropy over the logits of a tile (all classes in its 16 columns): labels, gradient at the logits [M][ld], loss per row
struct LoneCe { const int32_t *labels; void *dz; float *row_loss; int classes; };
template <typename T, bool CE, class LA, class LB>
__device__ __forceinline__ void lone_tile(LoneShared &sh, const LA &la, const LB &lb, const Epilogue &ep, int M, int N, int K, int tiles_n, int block,
                                          const LoneCe &ce)
{
    auto &part = sh.part;
    auto &sums = sh.sums;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    const int tm = block / tiles_n, tn = block - tm * tiles_n;
    const __amdgpu_buffer_rsrc_t ra = la.op.rsrc(), rb = lb.op.rsrc();
    const unsigned oa = row_offset(la, tm * 16 + (lane & 15)), ob = row_offset(lb, tn * 16 + (lane & 15));
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    Frag<T> fa, fb;
    int k = wave * 32 + 8 * (lane >> 4);
    load_piece(fa, la, ra, oa, k);
    load_piece(fb, lb, rb, ob, k);
    for (int k0 = wave * 32; k0 < K; k0 += waves * 32) {
        Frag<T> na, nb;
        k += waves * 32;
        load_piece(na, la, ra, oa, k);   // past K: zeros
        load_piece(nb, lb, rb, ob, k);
        mma16(acc, fb, fa);
        fa = na; fb = nb;
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (tid >= 64) return;
    // lane: row lane % 16, columns 4 * (lane / 16) ..
    f32x4 v = part[0][lane];
    for (int w = 1; w < waves; ++w) v = v + part[w][lane];
    if (ep.upd_w) {
        const int m = tm * 16 + (lane & 15), n0 = tn * 16 + 4 * (lane >> 4);
        if (m < M && n0 < N) {
            const long p = (long)m * ep.ld + n0;
            const f32x4 a = ep.upd_acc && !ep.upd_acc_first ? *reinterpret_cast<const f32x4 *>(__builtin_assume_aligned(ep.upd_acc + p, 16)) : f32x4{};
            push4<T>(ep, p, v, *reinterpret_cast<const f32x4 *>(__builtin_assume_aligned(ep.upd_w + p, 16)),
                     *reinterpret_cast<const f32x4 *>(__builtin_assume_aligned(ep.upd_v + p, 16)), a);
        }
        return;
    }
    *reinterpret_cast<f32x4 *>(&sums[lane & 15][4 * (lane >> 4)]) = v;
    __builtin_amdgcn_wave_barrier();   // one wave: its LDS accesses keep their order
    if constexpr (CE) {
        // four rows at a time, a lane per column; sums and comparisons in the order of softmax_ce_kernel
        const int c = lane & 15;
        const float bias = c < ep.bias_n ? to_f32(static_cast<const T *>(ep.bias)[c]) : 0.f, inv_b = 1.f / (float)M;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = q * 4 + (lane >> 4), m = tm * 16 + row;
            const float z = sums[row][c] + bias;
            float mx = c < ce.classes ? z : -INFINITY;
            for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
            float sum = c < ce.classes ? expf(z - mx) : 0.f;
            for (int o = 8; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
            const float lse = mx + logf(sum);
            const int label = m < M ? ce.labels[m] : 0;
            const bool label_ok = (unsigned)label < (unsigned)ce.classes;   // otherwise the row's loss is NaN and dz the plain softmax / M
            const float zl = __shfl(z, (lane & 48) + (label & 15), 64);
            if (m >= M || c >= N) continue;
            static_cast<float *>(ep.out)[(long)m * ep.ld + c] = z;
            static_cast<T *>(ce.dz)[(long)m * ep.ld + c] = (T)(c < ce.classes ? (expf(z - lse) - (c == label ? 1.f : 0.f)) * inv_b : 0.f);
            if (c == 0) ce.row_loss[m] = label_ok ? lse - zl : __builtin_nanf("");
        }
        return;
    }
    if (lane >= 32) return;
    const int m = tm * 16 + (lane >> 1), n0 = tn * 16 + 8 * (lane & 1);
    if (m >= M || n0 >= N) return;
    float o[8], bias8[8];
    load_bias8<T>(ep, n0, bias8);
#pragma unroll
    for (int r = 0; r < 8; ++r) o[r] = sums[lane >> 1][8 * (lane & 1) + r];
    epilogue8<T>(ep, m, n0, o, bias8);
}
template <typename T, class LA, class LB>
__global__ __launch_bounds__(64 * kLoneWaves) void lone_kernel(LA la, LB lb, Epilogue ep, int M, int N, int K, int tiles_n)
{
    __shared__ LoneShared sh;
    lone_tile<T, false>(sh, la, lb, ep, M, N, K, tiles_n, (int)blockIdx.x, LoneCe{});
}
// A last layer of up to 16 classes together with the softmax cross-entropy on top of it.
template <typename T>
__global__ __launch_bounds__(64 * kLoneWaves) void lone_ce_kernel(PlainK<T> la, PlainK<T> lb, Epilogue ep, int M, int N, int K, LoneCe ce)
{
    __shared__ LoneShared sh;
    lone_tile<T, true>(sh, la, lb, ep, M, N, K, 1, (int)blockIdx.x, ce);
}
// A weight gradient and a data gradient in one launch: neither waits for the other.  Each of these launches is 4 us or more of a pass whatever it
// computes: a step of the 28 x 28 net (8 images, fp32) 52 -> 43 us in 9 launches instead of 12, of the 32 x 32 net 230 -> 217 (fp32, 128
// images) and 158 -> 140 (bf16, 93 images, 27 -> 21), with the softmax in the kernel above and the partial sums of the filter gradients added
// up beside the pools' and the bias gradients' kernels.
template <typename T>
__global__ __launch_bounds__(64 * kLoneWaves) void lone_pair_kernel(LonePair<T> p)
{
    __shared__ LoneShared sh;
    if ((int)blockIdx.x < p.w_blocks) lone_tile<T, false>(sh, p.wa, p.wb, p.w_ep, p.w_m, p.w_n, p.w_k, p.w_tiles_n, (int)blockIdx.x, LoneCe{});
    else lone_tile<T, false>(sh, p.da, p.db, p.d_ep, p.d_m, p.d_n, p.d_k, p.d_tiles_n, (int)blockIdx.x - p.w_blocks, LoneCe{});
}

// gemm_kernel with the waves of a workgroup in two roles: Cfg::NT / 64 waves read
// fragments and multiply (wave tiles of 64 x 64), four more fetch both operands and move them into LDS.  Step t of
// a fetching wave: after the barrier, tile t+1 (fetched two steps ago) goes from its register set into the LDS stage
// that was multiplied in step t-1, and the set is refilled with tile t+3.
constexpr int kFetchThreads = 256;
template <typename T, class Cfg, class LA, class LB>
__global__ __launch_bounds__(Cfg::NT + kFetchThreads, Cfg::MINB) void gemm_ws_kernel(LA la, LB lb, Epilogue ep, int M, int N, int nkt, int kt_per_split,
                                                                           int tiles_m, int tiles_n, float *ws)
{
    constexpr int BK = Geo<T>::BK, BM = Cfg::BM, BN = Cfg::BN, NT = Cfg::NT, MB = Cfg::MB, NB = Cfg::NB, NP = kFetchThreads;
    constexpr int TA = LA::kTrans ? TransTile<T, BM>::BYTES : BM * 128, TB = LB::kTrans ? TransTile<T, BN>::BYTES : BN * 128;
    __shared__ uint4 smem[2 * (TA + TB) / 16];   // two stages of A and B tiles; reused to stage the output
    uint4 (*sA)[TA / 16] = reinterpret_cast<uint4 (*)[TA / 16]>(smem);
    uint4 (*sB)[TB / 16] = reinterpret_cast<uint4 (*)[TB / 16]>(smem + 2 * TA / 16);
    const int tid = threadIdx.x;
    int bid;
    {
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = blockIdx.x & 7;
        bid = x * q + (x < r ? x : r) + (blockIdx.x >> 3);
    }
    const int tn = bid % tiles_n; bid /= tiles_n;
    const int tm = bid % tiles_m;
    const int split = bid / tiles_m;
    const int kt0 = split * kt_per_split;
    const int nt = min(nkt, kt0 + kt_per_split) - kt0;   // K tiles of this workgroup (>= 1)

    if (tid >= NT) {
        const int ptid = tid - NT;
        Stage<T, LA, BM, NP, 2> stA;
        Stage<T, LB, BN, NP, 2> stB;
        stA.init(la, tm * BM, kt0 * BK, ptid, 0);
        stB.init(lb, tn * BN, kt0 * BK, ptid, NP / 2);
        stA.template load<0>(la); stB.template load<0>(lb);
        stA.template load<1>(la); stB.template load<1>(lb);
        stA.template store<0>(sA[0], ptid); stB.template store<0>(sB[0], ptid);
        stA.template load<0>(la); stB.template load<0>(lb);
        for (int t = 0; t < nt; t += 2) {
            __syncthreads();
            if (t + 1 < nt) { stA.template store<1>(sA[1], ptid); stB.template store<1>(sB[1], ptid); }
            stA.template load<1>(la); stB.template load<1>(lb);   // past the last tile this fetches zeros
            if (t + 1 < nt) {
                __syncthreads();
                if (t + 2 < nt) { stA.template store<0>(sA[0], ptid); stB.template store<0>(sB[0], ptid); }
                stA.template load<0>(la); stB.template load<0>(lb);
            }
        }
        // A wave that has ended no longer counts at the barriers of the output phase.  (Letting these waves help to take
        // the tile out of LDS makes the filter gradient 3.5 % slower.)
        return;
    }

    f32x16 acc[NB][MB];
    static_for<0, NB>([&](auto i) ASGD_INLINE { static_for<0, MB>([&](auto j) ASGD_INLINE { acc[i][j] = f32x16{}; }); });
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = (wave % Cfg::WAVES_M) * (BM / Cfg::WAVES_M), wn = (wave / Cfg::WAVES_M) * (BN / Cfg::WAVES_N);
    FragOff<T, LA::kTrans, BM> foA;
    FragOff<T, LB::kTrans, BN> foB;
    foA.init(wm, lane);
    foB.init(wn, lane);
    const bool busy = __builtin_amdgcn_readfirstlane((tm * BM + wm < M && tn * BN + wn < N) ? 1 : 0) != 0;
    float bias8[8];
    load_bias8<T>(ep, tn * BN + (tid % (BN / 8)) * 8, bias8);
    for (int t = 0; t < nt; t += 2) {
        __syncthreads();
        if (busy) compute_tile<T, MB, NB>(sA[0], sB[0], acc, foA, foB);
        if (t + 1 < nt) {
            __syncthreads();
            if (busy) compute_tile<T, MB, NB>(sA[1], sB[1], acc, foA, foB);
        }
    }
    output_tile<T, Cfg, (int)sizeof(smem)>(smem, acc, ep, tm, tn, split, M, N, ws, bias8, tid, wm, wn);
}

// The barrier of a wave that has buffer loads in flight that write LDS directly: its own LDS stores are waited for, the
// buffer loads are not (__syncthreads carries a release fence, for which the compiler drains every load that writes LDS);
// the "memory" clobber keeps the compiler from moving LDS accesses across it.
typedef __attribute__((address_space(3))) void lds_void;
__device__ __forceinline__ void barrier_keep_loads() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ------------------------------------------------------------------ first-layer convolution from staged image rows
// The window-row form of a first convolution (few input channels: a window row (kx, c) is one contiguous run of the
// bordered, channel-last image; K = (ky, j) with j over the padded run) has a short reduction (440 for 11 x 11 x 3)
// and a huge number of rows, so the tile engine above spends most of its time outside its seven-step K loop: every
// one of its 3025 workgroups fetches the same filters again, gathers an im2col tile that repeats every input element
// 7.6 times, and pays a head and an output phase.  This kernel keeps the whole filter bank in LDS for the lifetime
// of a workgroup (one per CU), walks over tiles of 128 output pixels of one image, and takes the A fragments
// straight from the image rows the tile needs (a contiguous block of the staged image, copied to LDS as it is): a
// lane's 8 consecutive K elements are 16 contiguous bytes of a window row, at byte offset
// (oy * stride + ky) * row_bytes + ox * stride * pixel_bytes + 2 j of the block.  There is no barrier inside the K
// loop.  Waves 0-3 multiply 64 x 32 blocks of the 128 x 96 tile, waves 4-7 32 x 32 blocks, which gives every SIMD
// three MFMA blocks.  The block of the next tile is fetched during the K loop of the current one; the output goes
// through LDS (the finished tile's block) so that a pixel's channels leave as 16-byte pieces.
struct RowsConv {
    Operand x; unsigned rowb, imgb;        // staged image: bytes per row (a multiple of 16) and per image
    unsigned pixstep;                      // bytes between the window origins of neighbouring output pixels (a multiple of 8)
    int Ho, Wo, stride, kh, KW, K;         // K = kh * KW; KW a multiple of 8
    int tiles_per_image, total, npix;      // npix = Ho * Wo
    Operand w; unsigned ldw;               // filters [N][K], bytes per row
    FastDiv dWo, dtpi, dKW;
};
constexpr int kRowsBM = 128, kRowsBN = 96, kRowsChunks = 7, kRowsPatchBytes = 32256, kRowsOutPitch = 208;

__global__ __launch_bounds__(512, 2) void conv_rows_kernel(RowsConv a, Epilogue ep, int N)
{
    typedef bf16_t T;
    constexpr int BM = kRowsBM, BN = kRowsBN, KC = kRowsChunks, PB = kRowsPatchBytes;
    constexpr int WBYTES = KC * BN * 128;                    // filters: [chunk][row][8 slots of 16 bytes], slots swizzled with the row
    __shared__ uint4 smem[(WBYTES + 2 * PB + 256) / 16];
    char *sW = reinterpret_cast<char *>(smem);
    char *sP = sW + WBYTES;                                  // two blocks of image rows
    constexpr unsigned kZero = (unsigned)(2 * PB);           // 256 bytes of zeros behind them (relative to sP)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lrow = lane & 31, half = lane >> 5;

    // ---- filters into LDS, once
    {
        const __amdgpu_buffer_rsrc_t rs = a.w.rsrc();
        for (int p = tid; p < KC * BN * 8; p += 512) {
            const int slot = p & 7, row = (p >> 3) % BN, chunk = (p >> 3) / BN;
            const int k = chunk * 64 + slot * 8;
            const unsigned off = (row < N && k < a.K) ? (unsigned)row * a.ldw + (unsigned)k * 2u : kInv;
            *reinterpret_cast<uint4 *>(sW + (chunk * BN + row) * 128 + ((slot ^ swz(row)) * 16)) = buf_ld16(rs, off);
        }
        if (tid < 16) *reinterpret_cast<uint4 *>(sP + kZero + tid * 16) = make_uint4(0u, 0u, 0u, 0u);
    }
    // ---- this wave's part of the tile
    const bool big = wave < 4;                               // 64 x 32 (two row blocks) or 32 x 32
    const int wm = big ? (wave & 1) * 64 : (wave - 4) * 32, wn = big ? (wave >> 1) * 32 : 64;
    FragOff<T, false, BN> foB;
    foB.init(wn, lane);
    // bias of this lane's 16 output columns: n = wn + 8 g + 4 half + j
    float bias[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int n = wn + 8 * (q >> 2) + 4 * half + (q & 3);
        bias[q] = (ep.bias && n < ep.bias_n) ? to_f32(static_cast<const T *>(ep.bias)[n]) : 0.f;
    }
    const __amdgpu_buffer_rsrc_t xrs = a.x.rsrc();
    // tile v of this workgroup -> (image, first pixel, first output row), and the block of image rows it needs
    auto decode = [&](int v, int &img, int &p0, int &oy0) ASGD_INLINE {
        const int q = a.total >> 3, r = a.total & 7, xx = v & 7;
        const int t = xx * q + (xx < r ? xx : r) + (v >> 3);     // each XCD gets a contiguous range of tiles
        img = (int)fdiv((uint32_t)t, a.dtpi);
        p0 = (t - img * a.tiles_per_image) * BM;
        oy0 = (int)fdiv((uint32_t)p0, a.dWo);
    };
    uint4 pr[4];                                             // the next tile's block on its way: 4 pieces of 16 bytes per thread
    auto block_load = [&](int v) ASGD_INLINE {
        int img, p0, oy0;
        decode(v, img, p0, oy0);
        const int p1 = min(p0 + BM, a.npix) - 1;
        const int rows = ((int)fdiv((uint32_t)p1, a.dWo) - oy0) * a.stride + a.kh;
        const unsigned src = (unsigned)img * a.imgb + (unsigned)(oy0 * a.stride) * a.rowb, bytes = (unsigned)rows * a.rowb;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned o = (unsigned)(tid + j * 512) * 16u;
            pr[j] = buf_ld16(xrs, o < bytes ? src + o : kInv);
        }
    };
    auto block_store = [&](int buf) ASGD_INLINE {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((tid + j * 512) * 16 < PB) *reinterpret_cast<uint4 *>(sP + buf * PB + (tid + j * 512) * 16) = pr[j];
    };

    int v = blockIdx.x;
    block_load(v);
    block_store(0);
    __syncthreads();
    for (int it = 0; v < a.total; ++it, v += gridDim.x) {
        const int buf = it & 1;
        const bool more = v + (int)gridDim.x < a.total;
        if (more) block_load(v + gridDim.x);                 // arrives during the K loop
        int img, p0, oy0;
        decode(v, img, p0, oy0);
        // the lane's rows of A: byte offset of the window origin inside the block, or nothing for rows past the image
        unsigned abase[2];
        bool aval[2];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            const int p = p0 + wm + mb * 32 + lrow;
            aval[mb] = p < a.npix && (mb == 0 || big);
            const int oy = (int)fdiv((uint32_t)min(p, a.npix - 1), a.dWo), ox = min(p, a.npix - 1) - oy * a.Wo;
            abase[mb] = (unsigned)(buf * PB) + (unsigned)((oy - oy0) * a.stride) * a.rowb + (unsigned)ox * a.pixstep;
        }
        f32x16 acc[2];
        acc[0] = f32x16{}; acc[1] = f32x16{};
        // K position of this lane's 8-element piece: (ky, j), advancing by 16 elements per K step.  The fragments of
        // K step s + 2 are asked for before the MFMAs of step s (three sets of fragment registers): a wave has only
        // one or two MFMAs per step, too few to hide the LDS latency of the step after it.
        int ky = 0, j = half * 8;
        if (j >= a.KW) { j -= a.KW; ky = 1; }
        Frag<T> fb[3], fa[3][2];
        auto issue = [&](auto sidx) ASGD_INLINE {
            constexpr int S = decltype(sidx)::value, SET = S % 3;
            const bool kval = ky < a.kh;
            const unsigned koff = (unsigned)ky * a.rowb + (unsigned)j * 2u;
            fb[SET].v = *reinterpret_cast<const uint4 *>(sW + (S / 4) * (BN * 128) + foB.o[S % 4][0]);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                if (mb == 0 || big) {
                    const unsigned ad = (kval && aval[mb]) ? abase[mb] + koff : kZero;
                    const uint2 lo = *reinterpret_cast<const uint2 *>(sP + ad), hi = *reinterpret_cast<const uint2 *>(sP + ad + 8);
                    fa[SET][mb].v = make_uint4(lo.x, lo.y, hi.x, hi.y);
                }
            }
            j += 16;
            if (j >= a.KW) { j -= a.KW; ++ky; }
            if (j >= a.KW) { j -= a.KW; ++ky; }               // KW >= 8: at most two window rows per step
        };
        issue(std::integral_constant<int, 0>{});
        issue(std::integral_constant<int, 1>{});
        static_for<0, KC * 4>([&](auto sidx) ASGD_INLINE {
            constexpr int S = decltype(sidx)::value, SET = S % 3;
            if constexpr (S + 2 < KC * 4) issue(std::integral_constant<int, S + 2>{});
            mma(acc[0], fb[SET], fa[SET][0]);
            if (big) mma(acc[1], fb[SET], fa[SET][1]);
        });
        __syncthreads();                                     // every wave has read its fragments: the block becomes the output stage
        char *so = sP + buf * PB;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            if (mb == 0 || big) {
                const int row = wm + mb * 32 + lrow;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    union { bf16_t h[4]; uint2 u; } o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float x = acc[mb][4 * g + e] + bias[4 * g + e];
                        if (ep.relu) x = x > 0.f ? x : 0.f;
                        o.h[e] = (bf16_t)x;
                    }
                    *reinterpret_cast<uint2 *>(so + row * kRowsOutPitch + (wn + 8 * g + 4 * half) * 2) = o.u;
                }
            }
        }
        __syncthreads();
        {   // a pixel's N channels leave as 16-byte pieces: 12 pieces per row of the 96 columns
            const long pix0 = (long)img * a.npix + p0;
            const int valid = min(BM, a.npix - p0), pieces = N / 8;
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const int e = tid + r * 512, row = e / 12, piece = e - row * 12;
                if (row < valid && piece < pieces)
                    *reinterpret_cast<uint4 *>(static_cast<char *>(ep.out) + ((pix0 + row) * ep.ld + piece * 8) * 2) =
                        *reinterpret_cast<const uint4 *>(so + row * kRowsOutPitch + piece * 16);
            }
        }
        if (more) block_store(buf ^ 1);                      // the other block: its tile's output left an iteration ago
        __syncthreads();
    }
}


// ------------------------------------------------------------------ first-layer filter gradient from staged image rows
// dW[cout][(ky, j)] = sum over output pixels of dY[pixel][cout] * window row element (ky, j) of that pixel: the
// reduction runs over the pixels, of which there are hundreds of thousands, and the result is tiny (96 x 440).  The
// tile engine splits it 128 ways, multiplies a quarter of its 128 x 512 padded tiles for nothing and gathers the
// im2col operand from memory again for every column tile.  Here a persistent workgroup (one per CU) walks over tiles
// of whole output rows of one image (up to 112 pixels) and keeps the whole 96 x 448 result in the accumulators of six waves (two
// or three blocks of 32 K columns each, all three blocks of output channels: 96 or 144 accumulator registers).  Both operands
// are read with transposing LDS reads, in which every lane supplies its own address: the dY tile is stored pixel by
// pixel (256-byte lines, the 64-byte group index XOR-ed with the line so that the four lines of a read fall into
// different banks), and the window-row elements come straight out of the block of image rows the tile touches,
// copied to LDS as it is (lane's K line = pixel: the byte offset of its window origin; lane's row piece = four
// consecutive K columns: ky * row_bytes + 2 j).  Two more waves do nothing but bring in the image rows and the dY tiles
// of the tiles to come with buffer loads that write LDS directly, three buffers each and two tiles ahead (with one tile of
// lead the period of a tile was the issue time of its 64 loads plus their latency, 3.2 us against 1.3 us of MFMAs),
// one barrier per tile.  Every workgroup leaves one partial result; the ordered split-K reduction adds them and
// scatters to canonical order.
constexpr int kRowsWgBN = 448, kRowsWgTP = 112, kRowsWgIB = 22528, kRowsWgDB = kRowsWgTP * 256, kRowsWgGrid = 256;

// rpt: output rows per tile (rpt * Wo <= kRowsWgTP pixels); a.tiles_per_image = ceil(Ho / rpt)
__global__ __launch_bounds__(512, 2) void conv_rows_wgrad_kernel(RowsConv a, int rpt, Operand dy, unsigned ldyb, int M, float *ws)
{
    typedef bf16_t T;
    constexpr int TP = kRowsWgTP, IB = kRowsWgIB, DB = kRowsWgDB, NI = IB / 1024, ND = DB / 1024;
    static_assert(NI <= 31 && ND <= 31, "two tiles of one wave's loads fit the six-bit in-order wait counter");
    __shared__ uint4 smem[(3 * IB + 3 * DB) / 16];
    char *sP = reinterpret_cast<char *>(smem);          // three blocks of image rows
    char *sD = sP + 3 * IB;                             // three dY tiles: TP lines of 256 bytes
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto decode = [&](int v, int &img, int &r0) ASGD_INLINE {
        const int q = a.total >> 3, r = a.total & 7, xx = v & 7;
        const int t = xx * q + (xx < r ? xx : r) + (v >> 3);     // each XCD gets a contiguous range of tiles
        img = (int)fdiv((uint32_t)t, a.dtpi);
        r0 = (t - img * a.tiles_per_image) * rpt;                // first output row of the tile
    };

    if (wave >= 6) {
        // ---- the two fetching waves (wave 6: image rows, wave 7: dY): tile `it` goes to buffers it % 3, two tiles ahead of
        // the multiplying waves.  One wave can have 63 loads (63 KB) in flight, less than a tile period needs.
        const __amdgpu_buffer_rsrc_t xrs = a.x.rsrc(), drs = dy.rsrc();
        // dY: instruction i fills lines 4 i .. 4 i + 3; lane l: line 4 i + l / 16, physical 16-byte slot l % 16, which holds
        // logical slot ((l % 16 / 4) ^ (line & 3)) * 4 + l % 4 of the pixel's row (line & 3 = l / 16)
        const int dline = lane >> 4, dslot = ((((lane & 15) >> 2) ^ dline) << 2) | (lane & 3);
        const bool dcol = dslot * 8 < M;
        const bool rows_wave = wave == 6;
        auto issue = [&](int v, int buf) ASGD_INLINE {   // always NI (or ND) instructions: the wait below counts them
            int img, r0;
            decode(v, img, r0);
            const int rows_out = min(rpt, a.Ho - r0);
            if (rows_wave) {
                const unsigned src = (unsigned)img * a.imgb + (unsigned)(r0 * a.stride) * a.rowb;
                const unsigned bytes = (unsigned)((rows_out - 1) * a.stride + a.kh) * a.rowb;
#pragma unroll 2
                for (int i = 0; i < NI; ++i) {
                    const unsigned o = (unsigned)(i * 64 + lane) * 16u;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(xrs, (lds_void *)(sP + buf * IB + i * 1024), 16, (int)(o < bytes ? src + o : kInv), 0, 0, 0);
                }
            } else {
                const int valid = rows_out * a.Wo;
                const unsigned dsrc = (unsigned)(img * a.npix + r0 * a.Wo) * ldyb + (unsigned)dslot * 16u;
#pragma unroll 2
                for (int i = 0; i < ND; ++i) {
                    const int line = i * 4 + dline;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(drs, (lds_void *)(sD + buf * DB + i * 1024), 16,
                                                             (int)((dcol && line < valid) ? dsrc + (unsigned)line * ldyb : kInv), 0, 0, 0);
                }
            }
        };
        int v = blockIdx.x;
        const int g = (int)gridDim.x;
        issue(v, 0);
        if (v + g < a.total) issue(v + g, 1);
        int buf2 = 2;                                        // buffer of tile it + 2
        for (; v < a.total; v += g) {   // tile `it`
            // tile `it` has landed when at most the next tile's instructions are outstanding (the counter retires in order)
            if (v + g >= a.total) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else if (rows_wave) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NI) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ND) : "memory");
            barrier_keep_loads();                            // ... and the buffers of tile it - 1 have been read to the end
            if (v + 2 * g < a.total) issue(v + 2 * g, buf2);
            buf2 = buf2 == 2 ? 0 : buf2 + 1;
        }
        return;
    }

    // ---- multiplying waves, all three blocks of output channels each.  Waves 0, 1, 4, 5 (two to a SIMD) own two blocks of
    // 32 K columns, waves 2 and 3 (which share their SIMDs with the fetching waves) three: 12 / 12 / 9 / 9 MFMAs per
    // K step on the four SIMDs.
    const int b4 = lane >> 4, i16 = lane & 15, lrow = lane & 31, half = lane >> 5;
    // A (dY tile): lane supplies K line 8 (b4 / 2) + i16 / 4 (+ 4) of the K step, channels mb * 32 + 16 (b4 & 1) + 4 (i16 & 3) ..+3
    unsigned aoff[3];
    static_for<0, 3>([&](auto mb) ASGD_INLINE {
        aoff[mb] = (unsigned)((8 * (b4 >> 1) + (i16 >> 2)) * 256 + ((mb ^ (i16 >> 2)) << 6) + 32 * (b4 & 1) + 8 * (i16 & 3));
    });
    // B (image rows): lane supplies the pixel of the same K line and K columns n .. n + 3.  The window origins of the
    // tile's pixels relative to its block of rows are the same for every tile (a tile is whole output rows).
    const int tp = rpt * a.Wo;                           // pixels of a full tile
    unsigned org[TP / 16][2];
    static_for<0, TP / 16>([&](auto ks) ASGD_INLINE {
        static_for<0, 2>([&](auto h) ASGD_INLINE {
            const int p = min(ks * 16 + 8 * (b4 >> 1) + (i16 >> 2) + 4 * h, tp - 1);   // lines past the tile hold zeros in dY
            const int oy = (int)fdiv((uint32_t)p, a.dWo), ox = p - oy * a.Wo;
            org[ks][h] = (unsigned)(oy * a.stride) * a.rowb + (unsigned)ox * a.pixstep;
        });
    });
    typedef __attribute__((address_space(3))) short4v lds_s4;
    auto tr_read = [&](const char *p0, const char *p1) ASGD_INLINE -> Frag<T> {
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(p0));
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(p1));
        const uint2 x = __builtin_bit_cast(uint2, lo), y = __builtin_bit_cast(uint2, hi);
        Frag<T> f;
        f.v = make_uint4(x.x, x.y, y.x, y.y);
        return f;
    };
    auto body = [&](auto nbw, int nb0) ASGD_INLINE {     // this wave's NBW blocks of K columns start at block nb0
        constexpr int NBW = decltype(nbw)::value;
        unsigned coff[NBW];
        static_for<0, NBW>([&](auto nb) ASGD_INLINE {
            int n = (nb0 + nb) * 32 + 16 * (b4 & 1) + 4 * (i16 & 3);
            n = min(n, a.K - 4);                         // columns past K: any valid address (their sums are not stored)
            const int ky = (int)fdiv((uint32_t)n, a.dKW);
            coff[nb] = (unsigned)ky * a.rowb + (unsigned)(n - ky * a.KW) * 2u;
        });
        f32x16 acc[NBW][3];
        static_for<0, NBW>([&](auto i) ASGD_INLINE { static_for<0, 3>([&](auto j) ASGD_INLINE { acc[i][j] = f32x16{}; }); });
        int buf = 0;
        for (int v = blockIdx.x; v < a.total; v += gridDim.x) {
            __syncthreads();
            const char *pa = sD + buf * DB, *pb = sP + buf * IB;
            // all TP / 16 K steps, whatever the tile holds (lines past its pixels are zeros in dY); the fragments of step
            // ks + 1 are asked for before the MFMAs of step ks
            Frag<T> fa[2][3], fb[2][NBW];
            auto frags = [&](auto ks) ASGD_INLINE {
                constexpr int S = decltype(ks)::value, SET = S & 1;
                static_for<0, 3>([&](auto mb) ASGD_INLINE { fa[SET][mb] = tr_read(pa + aoff[mb] + S * 16 * 256, pa + aoff[mb] + S * 16 * 256 + 4 * 256); });
                static_for<0, NBW>([&](auto nb) ASGD_INLINE { fb[SET][nb] = tr_read(pb + org[S][0] + coff[nb], pb + org[S][1] + coff[nb]); });
            };
            frags(std::integral_constant<int, 0>{});
            static_for<0, TP / 16>([&](auto ks) ASGD_INLINE {
                constexpr int S = decltype(ks)::value, SET = S & 1;
                if constexpr (S + 1 < TP / 16) frags(std::integral_constant<int, S + 1>{});
                static_for<0, NBW>([&](auto nb) ASGD_INLINE { static_for<0, 3>([&](auto mb) ASGD_INLINE { mma(acc[nb][mb], fb[SET][nb], fa[SET][mb]); }); });
            });
            buf = buf == 2 ? 0 : buf + 1;
        }
        // this workgroup's partial result: ws[block][m][n], n < K
        float *o = ws + (size_t)blockIdx.x * (size_t)M * (size_t)a.K;
        static_for<0, NBW>([&](auto nb) ASGD_INLINE {
            static_for<0, 3>([&](auto mb) ASGD_INLINE {
                const int m = mb * 32 + lrow;
                static_for<0, 4>([&](auto g) ASGD_INLINE {
                    const int n = (nb0 + nb) * 32 + 8 * g + 4 * half;
                    if (m < M && n < a.K)
                        *reinterpret_cast<f32x4 *>(o + (size_t)m * a.K + n) = f32x4{acc[nb][mb][4 * g], acc[nb][mb][4 * g + 1], acc[nb][mb][4 * g + 2], acc[nb][mb][4 * g + 3]};
                });
            });
        });
    };
    if (wave == 2 || wave == 3) body(std::integral_constant<int, 3>{}, 8 + (wave - 2) * 3);
    else body(std::integral_constant<int, 2>{}, (wave < 2 ? wave : wave - 2) * 2);
}

template <typename T> __global__ __launch_bounds__(256) void splitk_reduce_kernel(Reduction r) { reduce_plain<T>(r.ws, r.splits, r.ep, r.M, r.N, blockIdx.x); }
template <typename T, int L> __global__ __launch_bounds__(256) void splitk_reduce_wide_kernel(Reduction r)
{
    __shared__ float part[4][8];
    reduce_wide<T, L>(r.ws, r.splits, r.ep, r.M, r.N, blockIdx.x, part);
}
__global__ __launch_bounds__(256) void splitk_reduce_filters_kernel(Reduction r)
{
    __shared__ float sums[kReduceLds];
    reduce_filters(r.ws, r.splits, r.ep, r.M, r.N, r.npos, r.cb, r.chunks, blockIdx.x, sums);
}

// the reduction that follows a split GEMM
static Reduction plan_reduction(const float *ws, int splits, const Epilogue &ep, int M, int N)
{
    const long groups = (long)M * (N / 8);
    Reduction r;
    r.ws = ws; r.splits = splits; r.ep = ep; r.M = M; r.N = N;
    // Lanes that share a group: a chip full of blocks, and hardly more lanes than partials.  (us: 320 groups of 512 partials 10.8 with
    // 32 lanes, 8.6 with 256; 40 of 98 7.0 with 8, 3.3 with 256; 800 of 248 6.4 with 32, 7.5 with 256; 3200 of 70 6.8 with 8, 6.4
    // with 32; 5280 of 256, the AlexNet-style first layer, 14 with 32.  Few partials leave some of the 32 lanes without one and are
    // no longer for it: 300 to 1000 groups of 16 3.7 with 8, 3.5 with 32; of 32 4.2 and 3.6; of 63 6.4 and 4.0; 2500 to 8000 groups of
    // 16 3.9 and 4.0 to 5.2.)
    if (splits >= 64 && groups < 512) r.lanes = 256;
    else if ((splits >= 192 && groups < 8192) || (splits >= 16 && groups < 1024) || (splits >= 64 && groups < 4096)) r.lanes = 32;
    else if (splits >= 16 && groups < 32768) r.lanes = 8;
    else if (ep.mode == 1) {
        r.lanes = 0;
        r.npos = ep.cw_kh * ep.cw_kw; r.cb = r.npos <= 9 ? 64 : r.npos <= 64 ? 32 : 8; r.chunks = (ep.cw_cinp + r.cb - 1) / r.cb;   // npos * cb <= kReduceLds
    }
    r.blocks = r.lanes == 0 ? (unsigned)(M * r.chunks) : (unsigned)((groups * r.lanes + 255) / 256);
    return r;
}
int launch_reduction(int dtype, const Reduction &r, hipStream_t s)
{
    const auto go = [&](auto t) {
        using T = decltype(t);
        const dim3 grid(r.blocks), all(256);
        if (r.lanes == 256) hipLaunchKernelGGL((splitk_reduce_wide_kernel<T, 256>), grid, all, 0, s, r);
        else if (r.lanes == 32) hipLaunchKernelGGL((splitk_reduce_wide_kernel<T, 32>), grid, all, 0, s, r);
        else if (r.lanes == 8) hipLaunchKernelGGL((splitk_reduce_wide_kernel<T, 8>), grid, all, 0, s, r);
        else if (r.lanes == 0) hipLaunchKernelGGL(splitk_reduce_filters_kernel, grid, dim3((unsigned)std::min(256, (r.npos * r.cb / 4 + 63) / 64 * 64)), 0, s, r);
        else hipLaunchKernelGGL((splitk_reduce_kernel<T>), grid, all, 0, s, r);
    };
    if (dtype == kBF16) go(bf16_t());
    else go(0.f);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
int splitk_reduce(int dtype, const float *ws, int splits, const Epilogue &ep, int M, int N, Reduction *later, hipStream_t s)
{
    const Reduction r = plan_reduction(ws, splits, ep, M, N);
    if (!later) return launch_reduction(dtype, r, s);
    *later = r;
    return 0;
}

// ------------------------------------------------------------------ host side
GemmPlan plan_gemm(long M, long N, long K, int dtype, int max_splits)
{
    const int BK = dtype == kBF16 ? (int)Geo<bf16_t>::BK : (int)Geo<float>::BK;
    const int BM = Cfg128::BM, BN = Cfg128::BN;
    const long tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    const long nkt = (K + BK - 1) / BK;
    // A single row of tiles with a moderate K (the FC layers at batch <= 128) is bound by the partial sums it
    // writes and re-reads: one workgroup per CU with a deeper K range each beats two with half of it.
    const long target = (M <= BM && nkt <= 256) ? 256 : 512;
    long splits = 1;
    if (max_splits > 1 && tiles < target) {
        splits = target / tiles;                  // never more workgroups than run at once: a second, nearly empty round would double the time
        if (splits > nkt / 4) splits = nkt / 4;   // at least four K tiles per split
        if (splits > max_splits) splits = max_splits;
        if (splits < 1) splits = 1;
    }
    if (splits > 1) {  // no empty split
        const long per = (nkt + splits - 1) / splits;
        splits = (nkt + per - 1) / per;
    }
    GemmPlan p;
    p.splits = (int)splits;
    p.ws_floats = splits > 1 ? (size_t)splits * (size_t)M * (size_t)N : 0;
    return p;
}

// Convolution over M pixels with N output columns.  Up to 32 columns in tiles of 128 x 32 (a tile of 128 columns leaves three of four
// waves without a column: 3 -> 32 channels 5 x 5 on 32 x 32 in fp32, 128 images 28 -> 18 us), and where those tiles are fewer than half the CUs
// and K is long, in K splits: the launch that adds them up costs 5 us, a K tile alone on a CU 0.6 (64 -> 32 channels 5 x 5 on 7 x 7 in
// fp32, 128 images, 31 us in 49 tiles of conv_direct, 16 + 4 in 10 splits), as far as the partial sums fit.  In bf16, too: passes with one
// such convolution, tiles of 32 / 128 columns, 16 -> 32 channels 3 x 3, 25 tiles 55 / 56 us, 1693 tiles 138 / 153; 256 -> 24 channels 1 x 1,
// 1875 tiles 268 / 281; at most 1.01 over 460 convolutions and unstrided data gradients of 1 to 1875 tiles.  Data gradients of strided
// convolutions (zoom: their stride) in bf16 are bound by the addresses of their gather, which the 512 threads of the tiles of 128
// columns work out faster where a CU has one tile, or two and a long K: 25 K tiles (5 x 5, stride 2, over 64 channels) 129 to 252 tiles
// 27 us in 128 columns, 32 here, 368 and 509 tiles 34.5 in both, 613 tiles 52 and 41; 49 K tiles 44 and 56, 58 and 61, 88 and 73.  us: the
// modelled time.
GemmPlan plan_conv(long M, long N, long K, int dtype, int zoom, size_t partials, double *us)
{
    GemmPlan p = plan_gemm(M, N, K, dtype, 1);
    if (N > 32) return p;
    p.bn = 32;
    const int BK = dtype == kBF16 ? (int)Geo<bf16_t>::BK : (int)Geo<float>::BK;
    const double mfma = dtype == kBF16 ? 0.1 : 0.43;
    const long tiles = (M + 127) / 128, nkt = (K + BK - 1) / BK;
    const long fit = (long)std::min(partials / ((size_t)M * (size_t)N), (size_t)32);
    const long most = tiles >= 128 ? 1 : std::max(1L, std::min(std::min(nkt / 4, fit), 512 / tiles));
    double best = 0;
    for (long splits = 1, per = nkt; splits <= most;) {
        const double t = 8.0 + rounds_us(tiles * splits, 4, [&](int r) { return std::max(0.6, mfma * r) * per; }) +
                         (splits > 1 ? 5.0 + 1.5e-6 * splits * M * N : 0.0);
        if (best == 0 || t < best) { p.splits = (int)splits; best = t; }
        if (per == 1) break;
        splits = (nkt + per - 2) / (per - 1);
        per = (nkt + splits - 1) / splits;
    }
    if (zoom > 1 && dtype == kBF16 && p.splits == 1 && tiles <= 512 && nkt > (tiles <= 256 ? 8 : 32)) p.bn = 128;
    p.ws_floats = p.splits > 1 ? (size_t)p.splits * (size_t)M * (size_t)N : 0;
    if (us) *us = best;
    return p;
}

// Filter gradient over K pixels: M output channels, N window columns.  Up to 64 channels in tiles of 32 or 64 rows (a tile of 128
// leaves the matrix cores of waves beyond the channels idle: 32 channels, 5 x 5 over 32, fp32, 28800 pixels 51 us there, 24 here; 3
// channels, 131072 pixels 73 and 15), and in the number of pixel ranges with the smallest modelled time, partial sums included; in
// fp32 a K tile is 16 or 32 MFMAs of 64 cycles a SIMD, in bf16 it is its latency.  As many partial sums as the tile of 128 would leave
// are always allowed, more as far as they fit.
GemmPlan plan_filter_grad(long M, long N, long K, int dtype, size_t partials)
{
    const GemmPlan wide = plan_gemm(M, N, K, dtype, 128);
    if (M > 64) return wide;
    GemmPlan p;
    p.bm = M <= 32 ? 32 : 64;
    const int BK = dtype == kBF16 ? (int)Geo<bf16_t>::BK : (int)Geo<float>::BK, per_cu = p.bm == 32 && dtype == kF32 ? 3 : 2;
    const double mfma = dtype == kBF16 ? 0.0 : p.bm == 32 ? 0.43 : 0.86, alone = dtype == kBF16 ? 0.35 : 0.6;
    const long tiles = (N + 127) / 128, nkt = (K + BK - 1) / BK;
    const long fit = (long)std::min(partials / ((size_t)M * (size_t)N), (size_t)512);
    const long most = std::max(1L, std::min(nkt / 2, std::min(std::max(fit, (long)wide.splits), 256 * per_cu / tiles)));
    double best = 0;
    for (long splits = 1, per = nkt; splits <= most;) {
        const double us = rounds_us(tiles * splits, per_cu, [&](int r) { return std::max(alone * (0.75 + 0.25 * r), mfma * r) * per; }) +
                          (splits > 1 ? 2.0 + 1.5e-6 * splits * M * N : 0.0);
        if (best == 0 || us < best) { p.splits = (int)splits; best = us; }
        if (per == 1) break;
        splits = (nkt + per - 2) / (per - 1);                    // the fewest with fewer tiles each, none of them empty
        per = (nkt + splits - 1) / splits;
    }
    p.ws_floats = p.splits > 1 ? (size_t)p.splits * (size_t)M * (size_t)N : 0;
    return p;
}

// Where lone_kernel runs: hardly any work, which every tile may fetch anew, and a K that eight waves are not long over (10 outputs
// over 125 000 inputs, 2 images: 222 us here, 95 in 32 K splits of the tiles of 128; both take about 10 us at 4096).
static bool lone_applies(long M, long N, long K) { return M * N * K <= 32L << 20 && ((M + 15) / 16) * ((N + 15) / 16) <= 1024 && K <= 4096; }

double lone_fc_wgrad_us(int dtype, long out, long in, long batch)
{
    if (lone_applies(out, in, batch)) return 0.0;
    const long tiles = ((out + Cfg128::BM - 1) / Cfg128::BM) * ((in + Cfg128::BN - 1) / Cfg128::BN);
    if (tiles >= 128) return 0.0;
    // a workgroup alone on its CU: us per K tile of 128 bytes
    return dtype == kBF16 ? 0.54 * ((batch + 63) / 64) : 2.06 * ((batch + 31) / 32);
}

template <typename T, class Cfg, class LA, class LB>
static int run_tile(const LA &la, const LB &lb, int M, int N, int K, const Epilogue &ep, const GemmPlan &plan, float *ws, hipStream_t s, Reduction *later)
{
    constexpr int BK = Geo<T>::BK, BM = Cfg::BM, BN = Cfg::BN;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int nkt = (K + BK - 1) / BK;
    int splits = plan.splits;
    if (splits > 1 && ws == nullptr) return -1;
    const int per = (nkt + splits - 1) / splits;
    splits = (nkt + per - 1) / per;
    const long blocks = (long)tiles_m * tiles_n * splits;
    if (blocks > 0x7fffffffL) return -1;
    // The convolution filter gradient runs with fetching and multiplying waves (gemm_ws_kernel: -2.6 % in bf16, -4 % in
    // fp32 for the class); the im2col forward gather of the first layer is 12 % slower that way (seven K tiles: the
    // head of a workgroup weighs more than its loop) and stays as it is.
    if constexpr (std::is_same<LB, GatherT<T>>::value)
        hipLaunchKernelGGL((gemm_ws_kernel<T, Cfg, LA, LB>), dim3((unsigned)blocks), dim3(Cfg::NT + kFetchThreads), 0, s, la, lb, ep, M, N, nkt,
                           per, tiles_m, tiles_n, splits > 1 ? ws : nullptr);
    else
        hipLaunchKernelGGL((gemm_kernel<T, Cfg, LA, LB>), dim3((unsigned)blocks), dim3(Cfg::NT), 0, s, la, lb, ep, M, N, nkt, per, tiles_m,
                           tiles_n, splits > 1 ? ws : nullptr);
    if (hipGetLastError() != hipSuccess) return -1;
    return splits > 1 ? splitk_reduce(sizeof(T) == 2 ? kBF16 : kF32, ws, splits, ep, M, N, later, s) : 0;
}

template <typename T, class LA, class LB>
static int run(const LA &la, const LB &lb, int M, int N, int K, const Epilogue &ep, const GemmPlan &plan, float *ws, hipStream_t s, Reduction *later = nullptr)
{
    if (M <= 0 || N <= 0 || K <= 0 || (N & 7)) return -1;
    if (la.op.bytes == 0 || lb.op.bytes == 0) return -1;   // an operand beyond the 1 GiB the 32-bit offsets cover
    // Measured on the AlexNet-style shapes: the 8-wave form (four waves per SIMD hide more latency) wins everywhere
    // except the convolution filter gradient, whose two transposing operands want wider wave tiles (gemm_ws_kernel).
    constexpr bool plain = (std::is_same<LA, PlainK<T>>::value || std::is_same<LA, PlainT<T>>::value) &&
                           (std::is_same<LB, PlainK<T>>::value || std::is_same<LB, PlainT<T>>::value);
    if constexpr (plain) {
        if (lone_applies(M, N, K)) {
            const int tiles_n = (N + 15) / 16, waves = std::min(kLoneWaves, (K + 31) / 32);
            hipLaunchKernelGGL((lone_kernel<T, LA, LB>), dim3((unsigned)((M + 15) / 16 * tiles_n)), dim3((unsigned)(64 * waves)), 0, s, la, lb, ep, M, N, K,
                               tiles_n);
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
    }
    if constexpr (std::is_same<LB, GatherT<T>>::value) {
        if (plan.bm == 32) return run_tile<T, Cfg32<T>>(la, lb, M, N, K, ep, plan, ws, s, later);
        if (plan.bm == 64) return run_tile<T, Cfg64>(la, lb, M, N, K, ep, plan, ws, s, later);
        return run_tile<T, Cfg128>(la, lb, M, N, K, ep, plan, ws, s, later);
    } else {
        if constexpr (!plain)
            if (plan.bn == 32) return run_tile<T, CfgN32>(la, lb, M, N, K, ep, plan, ws, s, later);
        return run_tile<T, Cfg128w8>(la, lb, M, N, K, ep, plan, ws, s, later);
    }
}

static Operand operand(const void *p, size_t bytes) { return Operand{p, bytes <= kMaxOperandBytes ? (unsigned)bytes : 0u}; }

template <typename T, bool WIDE> static GatherK<T, WIDE> make_gather_k(const Gather &g)
{
    GatherK<T, WIDE> l;
    l.op = operand(g.x, g.bytes);
    l.pix = g.pix ? (unsigned)g.pix : (unsigned)(g.C * sizeof(T)); l.rowb = g.rowb ? (unsigned)g.rowb : (unsigned)(g.W * g.C * sizeof(T));
    l.H = g.H; l.W = g.W; l.C = g.C; l.Ho = g.Ho; l.Wo = g.Wo; l.kh = g.kh; l.kw = g.kw;
    l.sm = g.sm; l.pad = g.pad; l.M = g.N * g.Ho * g.Wo;
    l.adv_px = (int)Geo<T>::BK / g.C; l.adv_c = (int)Geo<T>::BK % g.C;
    l.dWo = make_fastdiv(g.Wo); l.dHoWo = make_fastdiv(g.Ho * g.Wo); l.dC = make_fastdiv(g.C); l.dkw = make_fastdiv(g.kw);
    return l;
}
template <typename T> static GatherKS<T> make_gather_ks(const Gather &g)
{
    GatherKS<T> l;
    l.op = operand(g.x, g.bytes);
    l.pix = g.pix ? (unsigned)g.pix : (unsigned)(g.C * sizeof(T));
    l.H = g.H; l.W = g.W; l.C = g.C; l.Ho = g.Ho; l.Wo = g.Wo; l.kh = g.kh; l.kw = g.kw;
    l.sm = g.sm; l.ds = g.ds; l.pad = g.pad; l.M = g.N * g.Ho * g.Wo;
    l.dWo = make_fastdiv(g.Wo); l.dHoWo = make_fastdiv(g.Ho * g.Wo); l.dC = make_fastdiv(g.C); l.dkw = make_fastdiv(g.kw);
    return l;
}
template <typename T> static GatherT<T> make_gather_t(const Gather &g)
{
    GatherT<T> l;
    l.op = operand(g.x, g.bytes);
    l.pix = g.pix ? (unsigned)g.pix : (unsigned)(g.C * sizeof(T)); l.rowb = g.rowb ? (unsigned)g.rowb : (unsigned)(g.W * g.C * sizeof(T));
    l.H = g.H; l.W = g.W; l.C = g.C; l.Ho = g.Ho; l.Wo = g.Wo; l.kh = g.kh; l.kw = g.kw;
    l.sm = g.sm; l.pad = g.pad; l.M = g.N * g.Ho * g.Wo; l.Krows = g.kh * g.kw * g.C;
    l.dWo = make_fastdiv(g.Wo); l.dHo = make_fastdiv(g.Ho); l.dHoWo = make_fastdiv(g.Ho * g.Wo); l.dC = make_fastdiv(g.C); l.dkw = make_fastdiv(g.kw);
    return l;
}
// [rows][ld] with K contiguous / [K][ld] with the rows contiguous; the byte range ends with the last element used
template <typename T> static PlainK<T> make_plain_k(const void *p, long ld, int rows, int K)
{
    return PlainK<T>{operand(p, ((size_t)(rows - 1) * ld + K) * sizeof(T)), (unsigned)(ld * sizeof(T)), rows, K};
}
template <typename T> static PlainT<T> make_plain_t(const void *p, long ld, int rows, int K)
{
    return PlainT<T>{operand(p, ((size_t)(K - 1) * ld + rows) * sizeof(T)), (unsigned)(ld * sizeof(T)), rows, K};
}

// The window-row form of a first convolution in 16-bit data with up to 96 output columns runs conv_rows_kernel when
// the filter bank and the image rows of a tile fit its LDS layout; everything else takes the tile engine.
static bool rows_applies(const Gather &a, long ldb, int N, const Epilogue &ep, const GemmPlan &plan)
{
    const long K = (long)a.kh * a.C;
    if (!(a.kw == 1 && a.pad == 0 && a.ds == 1 && a.pix != 0 && a.rowb != 0 && a.C % 8 == 0 && ldb == K && K <= 64 * kRowsChunks)) return false;
    if (!(N > 64 && N <= kRowsBN && N % 8 == 0 && plan.splits == 1)) return false;
    if (!(a.rowb % 16 == 0 && ((size_t)a.sm * a.pix) % 8 == 0 && ((uintptr_t)a.x & 15) == 0 && a.bytes <= kMaxOperandBytes)) return false;
    if (!(ep.mode == 0 && !ep.drop && !ep.mask_src && !ep.out_f32 && ep.ld % 8 == 0 && ((uintptr_t)ep.out & 15) == 0)) return false;
    const long out_rows = std::min<long>(a.Ho, (kRowsBM + a.Wo - 1) / a.Wo + 1);      // output rows a run of 128 pixels can touch
    const long block = ((out_rows - 1) * a.sm + a.kh) * (long)a.rowb;
    return block <= kRowsPatchBytes && a.H >= (a.Ho - 1) * a.sm + a.kh;
}
static int run_rows(const Gather &a, const void *b, long ldb, int N, const Epilogue &ep, hipStream_t s)
{
    RowsConv r;
    r.x = operand(a.x, a.bytes);
    r.rowb = (unsigned)a.rowb; r.imgb = (unsigned)((size_t)a.H * a.rowb); r.pixstep = (unsigned)((size_t)a.sm * a.pix);
    r.Ho = a.Ho; r.Wo = a.Wo; r.stride = a.sm; r.kh = a.kh; r.KW = a.C; r.K = a.kh * a.C;
    r.npix = a.Ho * a.Wo;
    r.tiles_per_image = (r.npix + kRowsBM - 1) / kRowsBM;
    const long total = (long)a.N * r.tiles_per_image;
    if (total <= 0 || total > 0x7fffffffL) return -1;
    r.total = (int)total;
    r.w = operand(b, (size_t)N * ldb * sizeof(bf16_t)); r.ldw = (unsigned)(ldb * sizeof(bf16_t));
    r.dWo = make_fastdiv((uint32_t)a.Wo); r.dtpi = make_fastdiv((uint32_t)r.tiles_per_image); r.dKW = make_fastdiv((uint32_t)a.C);
    if (r.x.bytes == 0 || r.w.bytes == 0) return -1;
    // one workgroup per CU (its LDS holds the filter bank and two blocks of image rows); a multiple of 8 so that every
    // workgroup's tiles stay on its XCD's contiguous range
    const long grid = total < 256 ? total : 256;
    hipLaunchKernelGGL(conv_rows_kernel, dim3((unsigned)grid), dim3(512), 0, s, r, ep, N);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T>
static int gather_plain_t(const Gather &a, const void *b, long ldb, int N, const Epilogue &ep, const GemmPlan &plan, float *ws, hipStream_t s)
{
    const int K = a.kh * a.kw * a.C;
    if constexpr (sizeof(T) == 2) {
        if (rows_applies(a, ldb, N, ep, plan)) return run_rows(a, b, ldb, N, ep, s);
    }
    if (a.ds == 1 && a.kh * a.kw <= 32)
        return run<T>(make_gather_k<T, false>(a), make_plain_k<T>(b, ldb, N, K), a.N * a.Ho * a.Wo, N, K, ep, plan, ws, s);
    if (a.ds == 1)
        return run<T>(make_gather_k<T, true>(a), make_plain_k<T>(b, ldb, N, K), a.N * a.Ho * a.Wo, N, K, ep, plan, ws, s);
    return run<T>(make_gather_ks<T>(a), make_plain_k<T>(b, ldb, N, K), a.N * a.Ho * a.Wo, N, K, ep, plan, ws, s);
}
int gemm_gather_plain(int dtype, const Gather &a, const void *b, long ldb, int N, const Epilogue &ep, const GemmPlan &plan, float *ws, hipStream_t s)
{
    if (a.ds != 1 && a.sm != 1) return -1;
    if (a.kh > 15 || a.kw > 15) return -1;
    return dtype == kBF16 ? gather_plain_t<bf16_t>(a, b, ldb, N, ep, plan, ws, s) : gather_plain_t<float>(a, b, ldb, N, ep, plan, ws, s);
}

// Where fc_split runs: 16-bit data, up to 64 rows, more than one K split (as many as have K tiles; otherwise 1).  Its head says why.
static int fc_splits(int dtype, int M, int N, int K, const GemmPlan &plan)
{
    if (dtype != kBF16 || M <= 0 || M > 64 || N <= 0 || N % 8 || K <= 0 || lone_applies(M, N, K)) return 1;
    const int nkt = (K + Geo<bf16_t>::BK - 1) / Geo<bf16_t>::BK, per = (nkt + plan.splits - 1) / plan.splits;
    return (nkt + per - 1) / per;
}
int gemm_plain_plain(int dtype, const void *a, long lda, int M, const void *b, long ldb, int N, int b_rows, int K, const Epilogue &ep,
                     const GemmPlan &plan, float *ws, hipStream_t s)
{
    if (b_rows > N) return -1;
    const int splits = fc_splits(dtype, M, N, K, plan);
    if (splits > 1) {
        if (fc_split(false, a, lda, M, b, ldb, N, b_rows, K, splits, plan.stream, ws, s) != 0) return -1;
        return splitk_reduce(kBF16, ws, splits, ep, M, N, nullptr, s);
    }
    if (dtype == kBF16)
        return run<bf16_t>(make_plain_k<bf16_t>(a, lda, M, K), make_plain_k<bf16_t>(b, ldb, b_rows, K), M, N, K, ep, plan, ws, s);
    return run<float>(make_plain_k<float>(a, lda, M, K), make_plain_k<float>(b, ldb, b_rows, K), M, N, K, ep, plan, ws, s);
}

int gemm_plain_trans(int dtype, const void *a, long lda, int M, const void *bt, long ldb, int N, int K, const Epilogue &ep,
                     const GemmPlan &plan, float *ws, hipStream_t s)
{
    const int splits = fc_splits(dtype, M, N, K, plan);
    if (splits > 1) {
        if (fc_split(true, a, lda, M, bt, ldb, N, N, K, splits, plan.stream, ws, s) != 0) return -1;
        return splitk_reduce(kBF16, ws, splits, ep, M, N, nullptr, s);
    }
    if (dtype == kBF16)
        return run<bf16_t>(make_plain_k<bf16_t>(a, lda, M, K), make_plain_t<bf16_t>(bt, ldb, N, K), M, N, K, ep, plan, ws, s);
    return run<float>(make_plain_k<float>(a, lda, M, K), make_plain_t<float>(bt, ldb, N, K), M, N, K, ep, plan, ws, s);
}

// Where outer_kernel runs: plain fp32 sums (no push), stores of 16 bytes, and either a tile for every CU or hardly a loop: with few
// tiles the K loop is what takes the time, and gemm_kernel fetches two K tiles ahead.  Serial pass of three layers of 4096, 4096 and
// 1000 outputs, gemm_kernel / here: bf16 128 images 204 / 168 us, 256 images 261 / 228, 512 images 366 / 346; fp32 460 / 417, 760 / 720,
// 1337 / 1299.  Of 64 and 10 outputs over 576 inputs: bf16 128 images 56.0 / 54.7, 2048 images 96 / 102; fp32 512 images 104 / 109.
template <typename T> static bool outer_applies(int M, int N, int K, const Epilogue &ep, const GemmPlan &plan)
{
    if (ep.upd_w || plan.splits != 1 || ep.mode != 0 || !ep.out_f32 || ep.bias || ep.relu || ep.drop || ep.mask_src) return false;
    const long tiles = ((M + 127) / 128) * (long)((N + 127) / 128);
    if (lone_applies(M, N, K) || !(K <= 2 * (int)Geo<T>::BK || (tiles >= 256 && K <= 512))) return false;
    return M > 0 && N > 0 && K > 0 && N % 8 == 0 && ep.ld % 4 == 0 && ((uintptr_t)ep.out & 15) == 0;
}
template <typename T> static int run_outer(const PlainT<T> &la, const PlainT<T> &lb, int M, int N, int K, const Epilogue &ep, hipStream_t s)
{
    if (la.op.bytes == 0 || lb.op.bytes == 0) return -1;
    const long tiles_n = (N + 127) / 128, blocks = (long)((M + 127) / 128) * tiles_n;
    if (blocks > 0x7fffffffL) return -1;
    hipLaunchKernelGGL((outer_kernel<T>), dim3((unsigned)blocks), dim3(512), 0, s, la, lb, static_cast<float *>(ep.out), ep.ld, M, N, K, (int)tiles_n);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
// A push inside the kernel (fc_push, update_tile of gemm_kernel over two transposed plain operands, or lone_kernel): whole sums only,
// 16-byte rows and column groups in all buffers.
static bool push_is_valid(const Epilogue &ep, const GemmPlan &plan)
{
    if (!ep.upd_w) return true;
    uintptr_t al = (uintptr_t)ep.upd_w | (uintptr_t)ep.upd_v | (uintptr_t)ep.upd_acc | (uintptr_t)ep.out;
    if (ep.upd_copies < 0 || ep.upd_copies > kPushCopies) return false;
    for (int c = 0; c < ep.upd_copies; ++c) { if (!ep.upd_copy[c]) return false; al |= (uintptr_t)ep.upd_copy[c]; }
    return plan.splits == 1 && ep.mode == 0 && ep.upd_v && !(al & 15) && !(ep.ld & 7);
}
int gemm_trans_trans(int dtype, const void *at, long lda, int M, const void *bt, long ldb, int N, int K, const Epilogue &ep,
                     const GemmPlan &plan, float *ws, hipStream_t s)
{
    if (!push_is_valid(ep, plan)) return -1;
    if (ep.upd_w) {
        if (fc_push_applies(dtype, M, N, K, ep)) return fc_push(at, lda, M, bt, ldb, N, K, ep, s);
    }
    if (dtype == kBF16)
        return outer_applies<bf16_t>(M, N, K, ep, plan)
                   ? run_outer(make_plain_t<bf16_t>(at, lda, M, K), make_plain_t<bf16_t>(bt, ldb, N, K), M, N, K, ep, s)
                   : run<bf16_t>(make_plain_t<bf16_t>(at, lda, M, K), make_plain_t<bf16_t>(bt, ldb, N, K), M, N, K, ep, plan, ws, s);
    return outer_applies<float>(M, N, K, ep, plan) ? run_outer(make_plain_t<float>(at, lda, M, K), make_plain_t<float>(bt, ldb, N, K), M, N, K, ep, s)
                                                   : run<float>(make_plain_t<float>(at, lda, M, K), make_plain_t<float>(bt, ldb, N, K), M, N, K, ep, plan, ws, s);
}

static int lone_tiles(int M, int N) { return (M + 15) / 16 * ((N + 15) / 16); }
static int lone_waves(int K) { return std::min(kLoneWaves, (K + 31) / 32); }
template <typename T> static int launch_lone_pair(const FcGrads &w, const FcGrads &d, const Epilogue &we, const Epilogue &de, hipStream_t s)
{
    LonePair<T> p;
    p.wa = make_plain_t<T>(w.dy, w.ld_dy, w.out, w.batch); p.wb = make_plain_t<T>(w.x, w.ld_x, w.in, w.batch);
    p.w_ep = we; p.w_m = w.out; p.w_n = w.in; p.w_k = w.batch; p.w_tiles_n = (w.in + 15) / 16; p.w_blocks = lone_tiles(w.out, w.in);
    p.da = make_plain_k<T>(d.dy, d.ld_dy, d.batch, d.out); p.db = make_plain_t<T>(d.w, d.in, d.in, d.out);
    p.d_ep = de; p.d_m = d.batch; p.d_n = d.in; p.d_k = d.out; p.d_tiles_n = (d.in + 15) / 16;
    if (p.wa.op.bytes == 0 || p.wb.op.bytes == 0 || p.da.op.bytes == 0 || p.db.op.bytes == 0) return -1;
    const unsigned blocks = (unsigned)(p.w_blocks + lone_tiles(d.batch, d.in)), threads = (unsigned)(64 * std::max(lone_waves(w.batch), lone_waves(d.out)));
    hipLaunchKernelGGL(lone_pair_kernel<T>, dim3(blocks), dim3(threads), 0, s, p);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
bool fc_pair_applies(const FcGrads &w, const FcGrads &d)
{
    return lone_applies(w.out, w.in, w.batch) && lone_applies(d.batch, d.in, d.out) && w.in % 8 == 0 && d.in % 8 == 0;
}
int fc_pair(int dtype, const FcGrads &w, const FcGrads &d, const Epilogue &we, const Epilogue &de, hipStream_t s)
{
    if (!push_is_valid(we, GemmPlan())) return -1;
    return dtype == kBF16 ? launch_lone_pair<bf16_t>(w, d, we, de, s) : launch_lone_pair<float>(w, d, we, de, s);
}

bool fc_softmax_applies(long M, long N, long K) { return N <= 16 && N % 8 == 0 && lone_applies(M, N, K); }
int fc_softmax(int dtype, const void *a, long lda, int M, const void *b, long ldb, int N, int classes, int K, const Epilogue &ep, const int32_t *labels, void *dz,
               float *row_loss, hipStream_t s)
{
    const LoneCe ce{labels, dz, row_loss, classes};
    const dim3 grid((unsigned)((M + 15) / 16)), block((unsigned)(64 * lone_waves(K)));
    const auto go = [&](auto t) {
        using T = decltype(t);
        const PlainK<T> la = make_plain_k<T>(a, lda, M, K), lb = make_plain_k<T>(b, ldb, classes, K);
        if (la.op.bytes == 0 || lb.op.bytes == 0) return -1;
        hipLaunchKernelGGL(lone_ce_kernel<T>, grid, block, 0, s, la, lb, ep, M, N, K, ce);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    };
    return dtype == kBF16 ? go(bf16_t()) : go(0.f);
}

// The filter gradient of a first convolution in window-row form (16-bit data, up to 96 output channels, up to 448 K
// columns) runs conv_rows_wgrad_kernel when the image rows of a tile fit its LDS layout and the plan has the scratch
// for one partial result per workgroup.
static int rows_wgrad_rpt(const Gather &b) { return b.Wo > 0 && b.Wo <= kRowsWgTP ? std::min(b.Ho, kRowsWgTP / b.Wo) : 0; }   // output rows per tile
static long rows_wgrad_tiles(const Gather &b)
{
    const int rpt = rows_wgrad_rpt(b);
    return rpt > 0 ? (long)b.N * ((b.Ho + rpt - 1) / rpt) : 0;
}
size_t rows_wgrad_ws_floats(int dtype, int M, const Gather &b)
{
    const long K = (long)b.kh * b.C, tiles = rows_wgrad_tiles(b);
    if (dtype != kBF16 || b.kw != 1 || b.pad != 0 || b.ds != 1 || M > 96 || K > kRowsWgBN || tiles <= 0) return 0;
    return (size_t)std::min<long>(tiles, kRowsWgGrid) * (size_t)M * (size_t)K;
}
static bool rows_wgrad_applies(const void *at, long lda, int M, const Gather &b, const Epilogue &ep, const GemmPlan &plan, const float *ws)
{
    const long K = (long)b.kh * b.C;
    const int rpt = rows_wgrad_rpt(b);
    if (rpt <= 0) return false;
    if (!(b.kw == 1 && b.pad == 0 && b.ds == 1 && b.pix != 0 && b.rowb != 0 && b.C % 8 == 0 && K <= kRowsWgBN && K % 8 == 0)) return false;
    if (!(M > 0 && M <= 96 && M % 8 == 0 && lda >= M && (lda * 2) % 16 == 0 && ((uintptr_t)at & 15) == 0)) return false;
    if (!(b.rowb % 16 == 0 && ((size_t)b.sm * b.pix) % 8 == 0 && ((uintptr_t)b.x & 15) == 0 && b.bytes <= kMaxOperandBytes)) return false;
    if (!(ep.mode == 2 && ep.out_f32 && ws != nullptr && ((uintptr_t)ws & 15) == 0 && plan.ws_floats >= rows_wgrad_ws_floats(kBF16, M, b))) return false;
    if ((size_t)b.N * b.Ho * b.Wo * lda * 2 > kMaxOperandBytes) return false;
    const long block = ((long)(rpt - 1) * b.sm + b.kh) * (long)b.rowb;   // image rows of a tile
    return block <= kRowsWgIB && b.H >= (b.Ho - 1) * b.sm + b.kh && rows_wgrad_tiles(b) <= 0x7fffffffL;
}
static int run_rows_wgrad(const void *at, long lda, int M, const Gather &b, const Epilogue &ep, float *ws, Reduction *later, hipStream_t s)
{
    RowsConv r;
    const int rpt = rows_wgrad_rpt(b);
    r.x = operand(b.x, b.bytes);
    r.rowb = (unsigned)b.rowb; r.imgb = (unsigned)((size_t)b.H * b.rowb); r.pixstep = (unsigned)((size_t)b.sm * b.pix);
    r.Ho = b.Ho; r.Wo = b.Wo; r.stride = b.sm; r.kh = b.kh; r.KW = b.C; r.K = b.kh * b.C;
    r.npix = b.Ho * b.Wo;
    r.tiles_per_image = (b.Ho + rpt - 1) / rpt;
    r.total = (int)rows_wgrad_tiles(b);
    r.w = Operand{nullptr, 0u}; r.ldw = 0;
    r.dWo = make_fastdiv((uint32_t)b.Wo); r.dtpi = make_fastdiv((uint32_t)r.tiles_per_image); r.dKW = make_fastdiv((uint32_t)b.C);
    const Operand dy = operand(at, (size_t)b.N * r.npix * lda * sizeof(bf16_t));
    if (r.x.bytes == 0 || dy.bytes == 0) return -1;
    const int grid = r.total < kRowsWgGrid ? r.total : kRowsWgGrid;
    hipLaunchKernelGGL(conv_rows_wgrad_kernel, dim3((unsigned)grid), dim3(512), 0, s, r, rpt, dy, (unsigned)(lda * sizeof(bf16_t)), M, ws);
    return hipGetLastError() == hipSuccess ? splitk_reduce(kBF16, ws, grid, ep, M, r.K, later, s) : -1;
}

int gemm_trans_gather(int dtype, const void *at, long lda, int M, const Gather &b, const Epilogue &ep, const GemmPlan &plan, float *ws,
                      Reduction *later, hipStream_t s)
{
    if (b.ds != 1 || b.kh > 15 || b.kw > 15) return -1;
    if (dtype == kBF16 && rows_wgrad_applies(at, lda, M, b, ep, plan, ws)) return run_rows_wgrad(at, lda, M, b, ep, ws, later, s);
    const int K = b.N * b.Ho * b.Wo, N = b.kh * b.kw * b.C;
    if (dtype == kBF16) return run<bf16_t>(make_plain_t<bf16_t>(at, lda, M, K), make_gather_t<bf16_t>(b), M, N, K, ep, plan, ws, s, later);
    return run<float>(make_plain_t<float>(at, lda, M, K), make_gather_t<float>(b), M, N, K, ep, plan, ws, s, later);
}

}  // namespace asgd
