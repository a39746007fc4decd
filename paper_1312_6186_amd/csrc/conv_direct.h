// The convolution kernel for stride-1 layers whose output grid equals their input grid: forward passes, and data gradients
// as convolutions with flipped filters.  Instantiated per element type and epilogue in conv_direct_*.hip; conv_direct.hip
// says where it applies and with which tile.
//
// With channel-last storage the input pixel that output pixel m needs at window position (ky, kx) is pixel
// m + (ky - pad) * W + (kx - pad) of the flattened tensor, whenever it lies inside the image.  A workgroup owns 32 MB WM
// pixels and 32 NB WN output channels and walks over chunks of 16 KS input channels.  The run of input pixels that its
// output pixels need at ALL window positions (the patch) lies in LDS once per chunk, so that a window position is the same
// LDS read at a shifted address; a lane whose window position lies outside the image reads zeros kept behind the patch, in
// the same banks.  The filters never touch LDS: they are packed in the order in which the matrix cores take them (see
// direct_index), a wave's fragment of a K step is one 1 KB load from L2, LOOK window positions ahead of its use.  The patch
// of the next chunk arrives in the other half of LDS, one load per window position (see direct_pieces), so that a chunk (9 or
// 25 window positions) has one barrier.
//
// Why: with both operands in LDS (128 x 128 tiles, wave tiles of 64 x 64, a barrier per 64 channels of one window position)
// LDS reads and writes took as long as the MFMAs.  Here a wave tile of 64 x 64 reads half as much from LDS and writes
// next to nothing, and wave tiles up to 96 x 96 have room in the registers.  What bounds it: the MFMAs (1.88 PFLOP/s is what
// this chip sustains on random bf16 data from registers), then what a tile costs outside its loop (9 us of 37 for the
// 13 x 13 layers at batch 128).  At one wave per SIMD and tiles of 32 rows, the filter loads: L1 gives 64 bytes a clock.
// The order of instructions matters: the scheduler otherwise gathers the loads behind the MFMAs, hence the group barriers.
//
// us, before -> after, bf16, 128 images (two layers with 5 x 5 windows on 27 x 27, then 3 x 3 on 13 x 13; kernel alone,
// inside a step): 96 -> 256 channels 129 -> 104, 256 -> 384 44 -> 37, 384 -> 384 58 -> 49, 384 -> 256 53 -> 39; data
// gradients 256 -> 96 136 -> 92, 384 -> 256 53 -> 42, 384 -> 384 58 -> 54, 256 -> 384 41 -> 41.  32 images: 42 -> 36,
// 28 -> 19, 36 -> 25, 31 -> 21; 58 -> 50, 32 -> 22, 35 -> 26, 26 -> 20 (256 -> 96 alone 44, and 41 since it runs in 128 x 128).
//
// The groups of a grouped layer are column tiles of one launch (a group has other input channels and filters, the pixels are the
// same): a launch each leaves the CUs idle twice at its start and end.  One step of the two-column net, bf16, 128 images
// (2 x 48 -> 128, 192 -> 192 and 192 -> 128 channels): 1235 -> 1201 us.
#pragma once
#include "asgd_internal.h"
#include "mfma_common.h"

namespace asgd {

struct DirectConv {
    Operand x; unsigned pix;               // activations, bytes from one pixel to the next
    int H, W, C, kh, kw, pad, npos, M, N;  // npos = kh * kw; M: pixels of the tensor = rows of C
    int nchunks, npl;                      // channel chunks; patch loads per thread and chunk
    unsigned patch_bytes, patch_off2;      // one patch buffer; offset of the second one (0 if there is one chunk)
    Operand w; unsigned nblk_bytes; int nblks;   // packed filters: bytes of a block of 32 output columns, and their number
    int tiles_n, groups;                   // column tiles of a group; groups, whose channels (C in, N out) and filters follow each other
    unsigned xg_bytes, wg_bytes;           // from one group's channels of a pixel to the next group's, and of the packed filters
    FastDiv dW, dHW;
};

// bytes of LDS behind the patches: zeros for window positions outside the image
constexpr int kDirectZero = 512;

// Loads per thread that the patch of the next chunk may take.  The load of window position j goes to LDS at position j + 1, that
// of the last position in its last K step, ahead of the chunk's barrier.  With one K step per chunk that step has the store of
// the position before ahead of the barrier and issues its own load behind it, so a load there would never arrive.
constexpr int direct_pieces(int ks, int npos) { return ks == 1 ? npos - 1 : npos; }

template <typename T, int KS> struct DirectGeo {
    static constexpr int PIECES = KS * 16 * (int)sizeof(T) / 16;       // 16-byte pieces of a pixel's chunk
    static constexpr int SH = PIECES > 4 ? 3 : PIECES > 2 ? 2 : 1;     // log2 of the threads that copy a pixel
    static constexpr int PITCH = KS * 16 * (int)sizeof(T) + 16;        // an odd number of pieces: neighbouring pixels in different banks
    static constexpr int KSB = 16 * (int)sizeof(T);                    // bytes of a K step
    static_assert(PIECES <= 8, "chunk of at most 128 bytes");
};

// LDS by byte address: with the base of the array folded into an address once, a read's address needs no addition.
typedef __attribute__((address_space(3))) uint4 lds_uint4;
__device__ __forceinline__ unsigned lds_addr(const uint4 *p) { return (unsigned)(size_t)(const lds_uint4 *)p; }
__device__ __forceinline__ uint4 lds_ld16(unsigned a)
{
    const u32x4 v = *reinterpret_cast<const __attribute__((address_space(3))) u32x4 *>(a);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void lds_st16(unsigned a, const uint4 &v)
{
    *reinterpret_cast<__attribute__((address_space(3))) u32x4 *>(a) = u32x4{v.x, v.y, v.z, v.w};
}
__device__ __forceinline__ void direct_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <typename T, int MB, int NB, int WM, int WN, int KS, int LOOK, bool MASKED>
__global__ __launch_bounds__(64 * WM * WN, (MB * NB > 8 ? 1 : 2)) void conv_direct_kernel(DirectConv p, Epilogue ep)
{
    using G = DirectGeo<T, KS>;
    constexpr int NT = 64 * WM * WN, BM = 32 * MB * WM, BN = 32 * NB * WN;
    constexpr int PPL = NT >> G::SH, PITCH = G::PITCH;   // pixels per patch load of the workgroup
    constexpr int VPF = (int)sizeof(T) / 2;              // 16-byte vectors per fragment
    extern __shared__ __attribute__((aligned(256))) uint4 smem4[];
    const unsigned sm = lds_addr(smem4);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lrow = lane & 31, half = lane >> 5;
    int bid;
    {
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = blockIdx.x & 7;
        bid = x * q + (x < r ? x : r) + (blockIdx.x >> 3);
    }
    // a tile's place: rows, group, columns.  Found anew for the output: the scalar registers that kept it would be spilled into
    // vector registers, and tiles of 96 x 96 would lose the second workgroup of a CU (one step at 142 images 1495 -> 1521 us).
    int tm, grp, tn;
    auto place = [&](int b) ASGD_INLINE {
        const int row = p.tiles_n * p.groups, c = b - (tm = b / row) * row;
        grp = c / p.tiles_n; tn = c - grp * p.tiles_n;
    };
    place(bid);
    const int wm = (wave % WM) * (32 * MB), wn = (wave / WM) * (32 * NB);
    const int total = p.nchunks * p.npos;
    const unsigned zero_base = sm + p.patch_off2 + p.patch_bytes;   // a multiple of 256

    // ---- filters: block of 32 columns, K step by K step, 64 lanes x 8 elements each
    const __amdgpu_buffer_rsrc_t wrs = p.w.rsrc();
    unsigned wvo[NB];
    static_for<0, NB>([&](auto nb) ASGD_INLINE {
        const int blk = min(tn * (BN / 32) + wn / 32 + nb, p.nblks - 1);   // columns past N: any block (never stored)
        wvo[nb] = (unsigned)grp * p.wg_bytes + (unsigned)blk * p.nblk_bytes + (unsigned)lane * (16u * VPF);
    });
    Frag<T> b[LOOK * KS][NB];   // LOOK window positions ahead; set r holds positions r, r + LOOK, ... (npos % LOOK == 0)
    auto load_b = [&](auto set, auto ks, auto nb, int step) ASGD_INLINE {
        const unsigned so = (unsigned)(step * KS + ks) * (1024u * VPF);
        if constexpr (sizeof(T) == 2) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(wrs, (int)wvo[nb], (int)so, 0);
            b[set * KS + ks][nb].v = make_uint4(v.x, v.y, v.z, v.w);
        } else {
            static_for<0, 2>([&](auto h) ASGD_INLINE {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(wrs, (int)wvo[nb] + h * 16, (int)so, 0);
                b[set * KS + ks][nb].v[h] = make_uint4(v.x, v.y, v.z, v.w);
            });
        }
    };
    // ---- patch: load j of a thread is slot `slot` of pixel prow + j * PPL
    const __amdgpu_buffer_rsrc_t xrs = p.x.rsrc();
    const int slot = tid & ((1 << G::SH) - 1), prow = tid >> G::SH;
    const int gp0 = tm * BM - p.pad * p.W - p.pad + prow;
    const bool act = slot < G::PIECES;
    // offset of load j (pixel gp = gp0 + j * PPL); cok: the slot's channels exist and load j belongs to the patch
    auto patch_off = [&](int gp, unsigned off, bool cok) ASGD_INLINE -> unsigned { return (((unsigned)gp < (unsigned)p.M) & cok) ? off : kInv; };
    const unsigned pvo0 = (unsigned)gp0 * p.pix + (unsigned)grp * p.xg_bytes + (unsigned)slot * 16u, pvo_step = (unsigned)PPL * p.pix;
    const unsigned pst = sm + (unsigned)(prow * PITCH + slot * 16);
    static_for<0, LOOK>([&](auto r) ASGD_INLINE { static_for<0, KS>([&](auto ks) ASGD_INLINE { static_for<0, NB>([&](auto nb) ASGD_INLINE { load_b(r, ks, nb, r); }); }); });
    for (int j0 = 0; j0 < p.npl; j0 += 6) {
        uint4 r[6];
        static_for<0, 6>([&](auto j) ASGD_INLINE { r[j] = buf_ld16(xrs, patch_off(gp0 + (j0 + j) * PPL, pvo0 + (unsigned)(j0 + j) * pvo_step, act & (slot * (16 / (int)sizeof(T)) < p.C) & (j0 + j < p.npl))); });
        static_for<0, 6>([&](auto j) ASGD_INLINE { if (act && j0 + j < p.npl) lds_st16(pst + (unsigned)(j0 + j) * (PPL * PITCH), r[j]); });
    }
    if (tid < kDirectZero / 16) lds_st16(zero_base + tid * 16, make_uint4(0u, 0u, 0u, 0u));
    // The filters are cold in this XCD's L2 (a kernel of this step has written them) and every workgroup walks through them
    // in the same order, a few fetches ahead: each would wait for memory again.  So the workgroups of an XCD first touch
    // them together, every thread four lines of its workgroup's share (32 images: data gradients 35 -> 28 us, 62 -> 50 us).
    unsigned touch[4];
    {
        const unsigned per = gridDim.x >> 3 ? gridDim.x >> 3 : 1u, mine = blockIdx.x >> 3;
        const unsigned share = (p.w.bytes / min(per, 32u) + 127u) & ~127u;
        static_for<0, 4>([&](auto i) ASGD_INLINE {
            const unsigned o = (unsigned)(i * NT + tid) * 128u;
            touch[i] = __builtin_amdgcn_raw_buffer_load_b32(wrs, (int)(mine < 32u && o < share ? mine * share + o : kInv), 0, 0);
        });
    }
    float bias_v = 0.f;
    if (ep.bias && tid < BN && tn * BN + tid < ep.bias_n) bias_v = to_f32(static_cast<const T *>(ep.bias)[grp * p.N + tn * BN + tid]);

    // ---- this lane's rows: patch address at window position (0, 0), and the window positions inside the image
    unsigned abase[MB], amask[MB];
    static_for<0, MB>([&](auto mb) ASGD_INLINE {
        const int rr = wm + mb * 32 + lrow, m = tm * BM + rr;
        abase[mb] = sm + (unsigned)(rr * PITCH + half * (8 * (int)sizeof(T)));
        unsigned mask = 0;
        if (m < p.M) {
            const int n = (int)fdiv((uint32_t)m, p.dHW);
            const int rem = m - n * (p.H * p.W);
            const int y = (int)fdiv((uint32_t)rem, p.dW);
            const int y0 = y - p.pad, x0 = rem - y * p.W - p.pad;
            const int ylo = max(0, -y0), yhi = max(ylo, min(p.kh, p.H - y0));
            const int xlo = max(0, -x0), xhi = max(xlo, min(p.kw, p.W - x0));
            const unsigned xm = ((1u << xhi) - 1u) & ~((1u << xlo) - 1u);
            for (int a = ylo; a < yhi; ++a) mask |= xm << (a * p.kw);
        }
        amask[mb] = mask;
    });
    f32x16 acc[NB][MB];
    static_for<0, NB>([&](auto i) ASGD_INLINE { static_for<0, MB>([&](auto j) ASGD_INLINE { acc[i][j] = f32x16{}; }); });

    // A K step's fragments are asked for one K step ahead; the sets rotate, so that after KS steps set 0 is next again
    // (KS = 1 has one set and a copy).
    constexpr int NSET = KS == 1 ? 2 : KS % 2 ? 3 : 2;
    Frag<T> fa[NSET][MB];
    int pos = 0, kx = 0;
    unsigned shift = 0, rowshift = 0, buf = 0;   // shift of the current window position in bytes of patch
    auto addr = [&](auto mb) ASGD_INLINE -> unsigned {
        const unsigned a = abase[mb] + (shift + buf);
        return ((amask[mb] >> pos) & 1u) ? a : (a & 0xF0u) | zero_base;
    };
    auto read_a = [&](auto set, const unsigned (&a)[MB], auto ks) ASGD_INLINE {
        static_for<0, MB>([&](auto mb) ASGD_INLINE {
            if constexpr (sizeof(T) == 2) {
                fa[set][mb].v = lds_ld16(a[mb] + ks * G::KSB);
            } else {
                fa[set][mb].v[0] = lds_ld16(a[mb] + ks * G::KSB);
                fa[set][mb].v[1] = lds_ld16(a[mb] + ks * G::KSB + 16);
            }
        });
    };
    direct_barrier();
    unsigned a[MB];
    static_for<0, MB>([&](auto mb) ASGD_INLINE { a[mb] = addr(mb); });
    read_a(std::integral_constant<int, 0>{}, a, std::integral_constant<int, 0>{});
    uint4 pr = make_uint4(0u, 0u, 0u, 0u);   // the piece of the next patch that is on its way
    unsigned pdst;                       // where it goes in LDS
    const unsigned dump = zero_base + kDirectZero + (unsigned)tid * 16u;   // where pieces of no patch go

    // One window position.  LAST: the chunk's last one, after which the patch of the next chunk must be complete.
    // Everything is free of branches, so that the address arithmetic and the copying run in the shadow of the MFMAs.
    int gp = 0, pj = 0;                  // pixel of the next patch load, and its number
    unsigned pvo = 0, pso = 0;           // its offset in the tensor and in the other patch buffer
    bool pok = false, cok = false;       // there is a next chunk and this thread has a slot in it; the slot's channels exist (else zeros go there)
    auto body = [&](auto set, auto last, int step) ASGD_INLINE {
        constexpr bool LAST = decltype(last)::value;
        const int nstep = min(step + LOOK, total - 1);
        const unsigned obuf = buf ^ p.patch_off2;
        if constexpr (LAST) { pos = 0; kx = 0; shift = 0; rowshift = 0; buf = obuf; }
        else {
            ++pos; ++kx; shift += PITCH;
            const bool up = kx == p.kw;
            rowshift += up ? (unsigned)(p.W * PITCH) : 0u; shift = up ? rowshift : shift; kx = up ? 0 : kx;
        }
        unsigned na[MB];
        static_for<0, KS>([&](auto ks) ASGD_INLINE {
            constexpr int cur = KS == 1 ? 0 : ks % NSET, nxt = KS == 1 ? 1 : (ks + 1) % NSET;
            if constexpr (ks == KS - 1) {
                if constexpr (KS == 1) static_for<0, MB>([&](auto mb) ASGD_INLINE { na[mb] = addr(mb); });
                if constexpr (LAST) {
                    lds_st16(pdst, pr);
                    direct_barrier();
                }
                read_a(std::integral_constant<int, nxt>{}, na, std::integral_constant<int, 0>{});
            } else {
                read_a(std::integral_constant<int, nxt>{}, a, std::integral_constant<int, ks + 1>{});
            }
            if constexpr (ks == 0) {
                if constexpr (KS > 1) static_for<0, MB>([&](auto mb) ASGD_INLINE { na[mb] = addr(mb); });
                // the patch of the next chunk: what the step before asked for goes to LDS, the next loads are issued (KS = 1:
                // that of the last position belongs to no patch, see direct_pieces)
                if constexpr (!(LAST && KS == 1)) lds_st16(pdst, pr);
                pr = buf_ld16(xrs, patch_off(gp, pvo, cok));
                pdst = (pok & (pj < p.npl)) ? pso : dump;
                gp += PPL; pvo += pvo_step; pso += PPL * PITCH; ++pj;
            }
            static_for<0, NB>([&](auto nb) ASGD_INLINE {
                static_for<0, MB>([&](auto mb) ASGD_INLINE { mma(acc[nb][mb], b[set * KS + ks][nb], fa[cur][mb]); });
                load_b(set, ks, nb, nstep);
            });
            static_for<0, NB>([&](auto nb) ASGD_INLINE {
                static_for<0, MB>([&](auto mb) ASGD_INLINE {
                    __builtin_amdgcn_sched_group_barrier(0x8, sizeof(T) == 2 ? 1 : 8, 0);
                    if constexpr (nb == 0) __builtin_amdgcn_sched_group_barrier(0x100, VPF, 0);
                    __builtin_amdgcn_sched_group_barrier(0x6, 6, 0);
                });
                __builtin_amdgcn_sched_group_barrier(0x20, VPF, 0);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (KS == 1) static_for<0, MB>([&](auto mb) ASGD_INLINE { fa[0][mb] = fa[1][mb]; });
        static_for<0, MB>([&](auto mb) ASGD_INLINE { a[mb] = na[mb]; });
    };
    for (int ch = 0, step = 0; ch < p.nchunks; ++ch) {
        const int c = (ch + 1) * (KS * 16) + slot * (16 / (int)sizeof(T));
        pok = act & (ch + 1 < p.nchunks);
        cok = pok & (c < p.C);
        gp = gp0; pj = 0;
        pvo = pvo0 + (unsigned)(ch + 1) * (unsigned)(KS * G::KSB); pso = (buf ^ p.patch_off2) + pst;
        pdst = dump;
        for (int q = LOOK; q < p.npos; q += LOOK)
            static_for<0, LOOK>([&](auto r) ASGD_INLINE { body(r, std::false_type{}, step++); });
        static_for<0, LOOK - 1>([&](auto r) ASGD_INLINE { body(r, std::false_type{}, step++); });
        body(std::integral_constant<int, LOOK - 1>{}, std::true_type{}, step++);
    }

    // ---- output: each wave moves its tile through its own part of LDS, 32 rows at a time, so that a lane ends up with 8
    // consecutive columns of a row
    asm volatile("" : "+s"(bid));
    place(bid);
    asm volatile("" ::"v"(touch[0]), "v"(touch[1]), "v"(touch[2]), "v"(touch[3]));
    char *smp = reinterpret_cast<char *>(smem4);
    float *sBias = reinterpret_cast<float *>(smp + WM * WN * NB * 4096);
    direct_barrier();
    if constexpr (!MASKED) {
        if (tid < BN) sBias[tid] = bias_v;
        direct_barrier();
    }
    char *st = smp + wave * (NB * 4096);
    constexpr int ITEMS = 2 * NB;
    const bool linear = !ep.relu;
    T *out = static_cast<T *>(ep.out) + grp * p.N;
    const T *mask = static_cast<const T *>(ep.mask_src) + grp * p.N;
    static_for<0, MB>([&](auto mb) ASGD_INLINE {
        const int m0 = tm * BM + wm + mb * 32;
        Vec8<T> ms[MASKED ? ITEMS : 1];
        if constexpr (MASKED) {
            static_for<0, ITEMS>([&](auto i) ASGD_INLINE {
                const int idx = lane + 64 * i, row = idx / (NB * 4), c8 = idx % (NB * 4), m = m0 + row, n0 = tn * BN + wn + c8 * 8;
                if (m < p.M && n0 < p.N) {
                    const uint4 *mp = reinterpret_cast<const uint4 *>(mask + (long)m * ep.mask_ld + n0);
                    static_for<0, VPF>([&](auto h) ASGD_INLINE { reinterpret_cast<uint4 *>(&ms[i])[h] = mp[h]; });
                }
            });
        }
        static_for<0, NB>([&](auto nb) ASGD_INLINE {
            static_for<0, 4>([&](auto g) ASGD_INLINE {
                const int chunk = nb * 8 + 2 * g + half;
                *reinterpret_cast<float4 *>(st + lrow * (NB * 128) + ((chunk ^ (lrow & 7)) * 16)) =
                    make_float4(acc[nb][mb][4 * g], acc[nb][mb][4 * g + 1], acc[nb][mb][4 * g + 2], acc[nb][mb][4 * g + 3]);
            });
        });
        static_for<0, ITEMS>([&](auto i) ASGD_INLINE {
            const int idx = lane + 64 * i, row = idx / (NB * 4), c8 = idx % (NB * 4), m = m0 + row, nl = wn + c8 * 8, n0 = tn * BN + nl;
            const float4 lo = *reinterpret_cast<const float4 *>(st + row * (NB * 128) + (((2 * c8) ^ (row & 7)) * 16));
            const float4 hi = *reinterpret_cast<const float4 *>(st + row * (NB * 128) + (((2 * c8 + 1) ^ (row & 7)) * 16));
            float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            if constexpr (MASKED) {
                static_for<0, 8>([&](auto r) ASGD_INLINE { v[r] = to_f32(ms[i].e[r]) > 0.f ? v[r] * ep.mask_scale : 0.f; });
            } else {
                const float4 b0 = *reinterpret_cast<const float4 *>(sBias + nl), b1 = *reinterpret_cast<const float4 *>(sBias + nl + 4);
                v[0] += b0.x; v[1] += b0.y; v[2] += b0.z; v[3] += b0.w; v[4] += b1.x; v[5] += b1.y; v[6] += b1.z; v[7] += b1.w;
                static_for<0, 8>([&](auto r) ASGD_INLINE { v[r] = ((v[r] > 0.f) | linear) ? v[r] : 0.f; });
            }
            if (m < p.M && n0 < p.N) store8<T>(out + (long)m * ep.ld + n0, v);
        });
    });
}


// The tile shapes: number, blocks of 32 rows and of 32 columns per wave, waves along the rows and along the columns.
#define ASGD_DIRECT_TILES(X) \
    X(0, 2, 2, 2, 2) X(1, 4, 2, 2, 2) X(2, 3, 2, 2, 2) X(3, 1, 2, 2, 2) X(4, 2, 1, 2, 2) X(5, 2, 3, 2, 2) X(6, 3, 3, 2, 2) \
    X(7, 3, 3, 4, 1) X(8, 2, 3, 4, 1) X(9, 1, 3, 4, 1) X(10, 2, 1, 4, 1) X(11, 1, 1, 4, 1)
constexpr int kDirectTiles = 12;
// Which of them exist for an element size and a number of K steps per chunk: K steps of 64 or 32 bf16 channels (32 fp32)
// are the ones that real layers have; 48 or 16 channels get by with fewer shapes.
constexpr bool direct_has(int es, int tile, int ks)
{
    const bool few = tile == 0 || tile == 3 || tile == 4 || tile == 10 || tile == 11;
    if (es == 2) return ks == 4 || ks == 2 ? true : ks == 3 ? (few || tile == 1) : few;
    return ks == 2 ? (tile != 1 && tile != 5 && tile != 6) : ks == 1 && few;
}

template <typename T, int MB, int NB, int WM, int WN, int KS, bool MASKED>
static int launch_direct_tile(const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s)
{
    // Filters three window positions ahead where the registers are there for it (3 x 3 windows, small wave tiles: at 32
    // images 26 -> 21 us for 384 -> 256 channels); larger wave tiles compute long enough per position.
    if constexpr (sizeof(T) == 2 && MB * NB <= 4 && KS >= 2) {
        if (p.npos % 3 == 0) {
            hipLaunchKernelGGL((conv_direct_kernel<T, MB, NB, WM, WN, KS, 3, MASKED>), dim3(grid), dim3(64 * WM * WN), lds, s, p, ep);
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
    }
    hipLaunchKernelGGL((conv_direct_kernel<T, MB, NB, WM, WN, KS, 1, MASKED>), dim3(grid), dim3(64 * WM * WN), lds, s, p, ep);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
template <typename T, bool MASKED> static int launch_direct_t(int tile, int ks, const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s)
{
#define ASGD_DIRECT_CASE(V, MB, NB, WM, WN, KS) \
    if constexpr (direct_has((int)sizeof(T), V, KS)) { if (tile == V && ks == KS) return launch_direct_tile<T, MB, NB, WM, WN, KS, MASKED>(p, ep, grid, lds, s); }
#define ASGD_DIRECT_TILE(V, MB, NB, WM, WN) \
    ASGD_DIRECT_CASE(V, MB, NB, WM, WN, 4) ASGD_DIRECT_CASE(V, MB, NB, WM, WN, 3) ASGD_DIRECT_CASE(V, MB, NB, WM, WN, 2) ASGD_DIRECT_CASE(V, MB, NB, WM, WN, 1)
    ASGD_DIRECT_TILES(ASGD_DIRECT_TILE)
#undef ASGD_DIRECT_TILE
#undef ASGD_DIRECT_CASE
    return -1;
}
int launch_direct_bf16_fwd(int tile, int ks, const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s);
int launch_direct_bf16_bwd(int tile, int ks, const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s);
int launch_direct_f32_fwd(int tile, int ks, const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s);
int launch_direct_f32_bwd(int tile, int ks, const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s);

}  // namespace asgd
