// The push of a fully-connected layer's weights in the kernel that computes their gradient, 16-bit data: for every weight g is a sum over the
// minibatch, t = g + wd * w, v = mu * v - lr * t, w = w + v, and the new weights go to the replicas' copies.
//
// What bounds it is memory: 18 bytes a weight.  4096 x 9216 over 128 images take 125 us again and again (5.4 TB/s) and 138 after a copy of 1 GiB (4.9;
// the copy itself 5.2), in gemm_kernel 123 and 131.  One workgroup of four
// waves a CU is enough for that if loads never pause, and leaves most of the LDS and the registers of a CU to the kernels of the
// other stream: with tiles of 128 x 128 and two workgroups of 80 KB a CU (gemm_kernel) a data gradient finds no room
// until the whole push is over.  So a workgroup walks over tiles of 64 x 128, down a strip of columns whose inputs it keeps as
// fragments in registers; the rows' output gradients arrive one tile ahead, and the parameters and momenta of a tile (64 KB a
// workgroup) are on their way while the one before is stored.  Loads return in order, so a tile's output gradients are asked for
// ahead of its parameters: waiting for the former does not wait for the latter.  A wave owns 32 columns, a line of memory in every row, and
// turns its sums from the matrix cores' order into rows through 4 KB of LDS of its own, without a barrier.
// One step, gemm_kernel / here, all else the same: AlexNet-style net, 128 images 1276 / 1228 us, 256 images 2195 / 2143, two-column net 1173 / 1132.
// Workgroups 128, 192, 256, 320, 384, 512 on one box: alone 170, 134, 125, 161, 145, 128; the three steps 1337, 1273, 1266, 1317, 1294, 1291; 2174,
// 2246, 2212, 2254, 2232, 2236; 1223, 1172, 1162, 1190, 1183, 1173.  With half or a quarter of the parameters on their way it is 3 and 5 %
// slower alone, on a third stream, beside the filter gradients too, a step 1 %.  Ordinary parameter loads: fc_push_pays; ordinary stores beside
// convolutions 5 %; non-temporal stores of the copies 15 % alone.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "asgd_internal.h"
#include "mfma_common.h"

namespace asgd {

namespace {

constexpr int kPushBM = 64, kPushBN = 128;   // a tile: rows (outputs), columns (inputs); a wave owns 32 columns

struct FcPush {
    Operand a, b;                 // output gradients [K][lda], inputs [K][ldb]
    unsigned lda, ldb;            // bytes from one image to the next
    int M, N, K, tiles_m, total;  // total: tiles
    unsigned ld;                  // elements from one row of the parameters to the next
    float *w, *v, *out;
    bf16_t *copy[kPushCopies];
    int copies;
    float lr, mu, wd;
};

constexpr int kNt = 2;   // non-temporal
__device__ __forceinline__ f32x4 buf_ldf4(__amdgpu_buffer_rsrc_t rs, unsigned off)
{
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, kNt));
}
__device__ __forceinline__ void buf_stf4(__amdgpu_buffer_rsrc_t rs, unsigned off, f32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, (int)off, 0, kNt);
}
__device__ __forceinline__ uint32_t bf16_bits(uint32_t u)   // round to nearest even, NaN kept
{
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (u >> 16) | 0x0040u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ void push_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace

template <int KF, int R>   // K steps of 16 images; groups of 8 rows per set of parameters
__global__ __launch_bounds__(256, 2) void fc_push_kernel(FcPush p)
{
    constexpr int KL = KF * 16, LA = TransTile<bf16_t, kPushBM>::LINE, LB = TransTile<bf16_t, kPushBN>::LINE;
    constexpr int BCH = KF < 4 ? KF : 4;                      // K steps of the inputs that are staged at a time
    constexpr int A_BYTES = KL * LA, B_BYTES = BCH * 16 * LB;
    constexpr int SMEM = A_BYTES + 4 * 4096 > B_BYTES ? A_BYTES + 4 * 4096 : B_BYTES;
    constexpr int SUBS = 8 / R, PA = KL / 32, PB = BCH;                     // 16-byte pieces per thread
    __shared__ uint4 smem[SMEM / 16];
    char *sm = reinterpret_cast<char *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int bid;
    {
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = blockIdx.x & 7;
        bid = x * q + (x < r ? x : r) + (blockIdx.x >> 3);
    }
    int t = (int)((long)p.total * bid / gridDim.x);
    const int t1 = (int)((long)p.total * (bid + 1) / gridDim.x);
    if (t >= t1) return;
    int tn = t / p.tiles_m, tm = t - tn * p.tiles_m;

    // ---- inputs of this wave's 32 columns: fragments of all K, kept while the workgroup walks down the rows
    const __amdgpu_buffer_rsrc_t rb = p.b.rsrc(), ra = p.a.rsrc();
    Frag<bf16_t> fb[KF];
    FragOff<bf16_t, true, kPushBN> foB;
    foB.init(wave * 32, lane);
    auto load_inputs = [&]() ASGD_INLINE {
        const int piece = tid & 15, line = tid >> 4, n0 = tn * kPushBN + piece * 8;
        const unsigned off = n0 < p.N ? (unsigned)n0 * 2u : kInv;
        static_for<0, KF / BCH>([&](auto c) ASGD_INLINE {
            uint4 r[PB];
            static_for<0, PB>([&](auto i) ASGD_INLINE {
                const int k = c * (BCH * 16) + i * 16 + line;
                r[i] = buf_ld16(rb, off + (k < p.K ? (unsigned)k * p.ldb : kInv));
            });
            push_barrier();
            static_for<0, PB>([&](auto i) ASGD_INLINE { *reinterpret_cast<uint4 *>(sm + (i * 16 + line) * LB + piece * 16) = r[i]; });
            push_barrier();
            static_for<0, BCH>([&](auto ks) ASGD_INLINE { fb[c * BCH + ks].template read<ks, 0>(sm, foB); });
        });
    };
    // ---- output gradients of a tile's rows: all of K, one tile ahead in registers
    uint4 st[PA];
    const int apiece = tid & 7, aline = tid >> 3;
    auto load_rows = [&](int tile, bool ok) ASGD_INLINE {
        const int m0 = tile * kPushBM + apiece * 8;
        const unsigned off = (m0 < p.M && ok) ? (unsigned)m0 * 2u : kInv;
        static_for<0, PA>([&](auto i) ASGD_INLINE {
            const int k = i * 32 + aline;
            st[i] = buf_ld16(ra, off + (k < p.K ? (unsigned)k * p.lda : kInv));
        });
    };
    FragOff<bf16_t, true, kPushBM> foA;
    foA.init(0, lane);
    // ---- parameters: block mb of a tile is 32 rows of this wave's columns; a lane owns 4 columns of the rows r * 8 + lane / 8
    f32x4 w[2][R], mo[2][R];
    const int piece = lane & 7, lrow8 = lane >> 3, col = wave * 32 + piece * 4;
    auto range = [&](int tm_, int tn_, bool ok) ASGD_INLINE -> unsigned {   // elements of a tile from its first one on
        return ok ? (unsigned)min(kPushBM, p.M - tm_ * kPushBM) * p.ld - (unsigned)tn_ * kPushBN : 0u;
    };
    auto rsrc4 = [&](float *base, long first, unsigned n) ASGD_INLINE { return Operand{base + first, n * 4u}.rsrc(); };
    auto voff = [&](int tn_, auto sub, auto r) ASGD_INLINE -> unsigned {
        const unsigned o = tn_ * kPushBN + col < p.N ? ((unsigned)lrow8 * p.ld + (unsigned)col) * 4u : kInv;
        return o + (unsigned)((sub * R + r) * 8) * p.ld * 4u;
    };
    auto load_params = [&](auto sub, int tm_, int tn_, bool ok) ASGD_INLINE {
        constexpr int set = sub % 2;
        const long first = (long)tm_ * kPushBM * p.ld + tn_ * kPushBN;
        const unsigned n = range(tm_, tn_, ok);
        const __amdgpu_buffer_rsrc_t rw = rsrc4(p.w, first, n), rv = rsrc4(p.v, first, n);
        static_for<0, R>([&](auto r) ASGD_INLINE { w[set][r] = buf_ldf4(rw, voff(tn_, sub, r)); });
        static_for<0, R>([&](auto r) ASGD_INLINE { mo[set][r] = buf_ldf4(rv, voff(tn_, sub, r)); });
    };

    load_inputs();
    load_rows(tm, true);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): nothing of this is in flight at the head of the loop
    load_params(std::integral_constant<int, 0>{}, tm, tn, true);
    load_params(std::integral_constant<int, 1>{}, tm, tn, true);
    for (;;) {
        push_barrier();
        static_for<0, PA>([&](auto i) ASGD_INLINE { *reinterpret_cast<uint4 *>(sm + (i * 32 + aline) * LA + apiece * 16) = st[i]; });
        push_barrier();
        f32x16 acc[2];
        acc[0] = f32x16{}; acc[1] = f32x16{};
        static_for<0, KF>([&](auto ks) ASGD_INLINE {
            Frag<bf16_t> fa[2];
            static_for<0, 2>([&](auto mb) ASGD_INLINE { fa[mb].template read<ks, mb>(sm, foA); });
            static_for<0, 2>([&](auto mb) ASGD_INLINE { mma(acc[mb], fb[ks], fa[mb]); });
        });
        const bool more = t + 1 < t1;
        const int ntm = tm + 1 == p.tiles_m ? 0 : tm + 1, ntn = tm + 1 == p.tiles_m ? tn + 1 : tn;
        load_rows(ntm, more);   // ahead of the parameters: waiting for these does not wait for those
        f32x4 *stg = reinterpret_cast<f32x4 *>(sm + A_BYTES) + wave * 256;
        const int lrow = lane & 31, half = lane >> 5;
        static_for<0, SUBS>([&](auto sub) ASGD_INLINE {
            constexpr int set = sub % 2, mb = sub * R / 4;
            if constexpr (sub * R % 4 == 0)
                static_for<0, 4>([&](auto g) ASGD_INLINE {
                    stg[lrow * 8 + ((2 * g + half) ^ (lrow & 7))] = f32x4{acc[mb][4 * g], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]};
                });
            const long first = (long)tm * kPushBM * p.ld + tn * kPushBN;
            const unsigned n = range(tm, tn, true);
            const __amdgpu_buffer_rsrc_t rw = rsrc4(p.w, first, n), rv = rsrc4(p.v, first, n);
            f32x4 g[R];
            static_for<0, R>([&](auto r) ASGD_INLINE { g[r] = stg[((sub * R % 4 + r) * 8 + lrow8) * 8 + (piece ^ lrow8)]; });
            static_for<0, R>([&](auto r) ASGD_INLINE {
                f32x4 wo = w[set][r], vo = mo[set][r];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float tt = __builtin_fmaf(p.wd, wo[e], g[r][e]);
                    const float vn = __builtin_fmaf(p.mu, vo[e], -(p.lr * tt));
                    vo[e] = vn;
                    wo[e] = wo[e] + vn;
                }
                buf_stf4(rw, voff(tn, sub, r), wo);
                buf_stf4(rv, voff(tn, sub, r), vo);
                w[set][r] = wo;
            });
            if (p.out) {
                const __amdgpu_buffer_rsrc_t ro = rsrc4(p.out, first, n);
                static_for<0, R>([&](auto r) ASGD_INLINE { buf_stf4(ro, voff(tn, sub, r), g[r]); });
            }
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            u32x2 h[R];
            static_for<0, R>([&](auto r) ASGD_INLINE {
                const f32x4 x = w[set][r];
                h[r].x = bf16_bits(__float_as_uint(x[0])) | (bf16_bits(__float_as_uint(x[1])) << 16);
                h[r].y = bf16_bits(__float_as_uint(x[2])) | (bf16_bits(__float_as_uint(x[3])) << 16);
            });
            for (int c = 0; c < p.copies; ++c) {
                const __amdgpu_buffer_rsrc_t rc = Operand{p.copy[c] + first, n * 2u}.rsrc();
                static_for<0, R>([&](auto r) ASGD_INLINE { __builtin_amdgcn_raw_buffer_store_b64(h[r], rc, (int)(voff(tn, sub, r) >> 1), 0, 0); });
            }
            if constexpr (sub + 2 < SUBS) load_params(std::integral_constant<int, sub + 2>{}, tm, tn, true);
            else load_params(std::integral_constant<int, sub + 2 - SUBS>{}, ntm, ntn, more);
        });
        if (!more) break;
        const bool strip = ntn != tn;
        ++t; tm = ntm; tn = ntn;
        if (strip) load_inputs();
    }
}

// What it is for is the room it leaves, to the kernels of the other stream; its loads, non-temporal in any case, find nothing in the caches.
// One step, gemm_kernel / here, us.  Convolutions below of 64 and 128 channels on 32 x 32 images: 16.8 M parameters, 64 images 230 / 231, 256 images
// 334 / 298; 33.6 M, 16 images 260 / 255, 256 images 415 / 380; the two-column net 697 / 655 at 32 images, 1173 / 1132 at 128.  With next to nothing below: 13 M
// 183 / 189, 19 M 204 / 215, 26 M 230 / 242 at 64 images, 34 M 255 / 254 at 16 and 291 / 278 at 128, 59 M 440 / 403 at 64: there only vectors far
// beyond the caches.  (Ordinary loads: 19 M 204, 59 M 471; convolutions below, 16.8 M, 256 images 316.)  On one stream the push of a small layer is
// faster here by itself: 2048 to 1000, cold caches, 16 / 13, hot 9.3 / 7.0.
// Beside other replicas' passes, eight updates, AlexNet-style net: 2 x 16 images 4759 / 4895, 4 x 32 5606 / 5643, 4 x 64 7010 / 7020, 4 x 96 8427 / 8388,
// 4 x 128 9872 / 9756; 19 M parameters with next to nothing below, 4 x 16 1212 / 1328.  An update of a replay that no other replica's gradient runs beside
// is a step: every gradient on the newest version, 2 x 16 images 5632 / 5594, 2 x 20 5758 / 5752, 2 x 26 6004 / 6065; 59 M 3219 / 2982; both kinds in one
// schedule, 4 x 16 (one update stale at most) 4959 / 4964, 4 x 32 5656 / 5628; 59 M 3053 / 2943.
bool fc_push_pays(size_t params, double conv_flops, long batch, bool one_stream, bool others)
{
    if (one_stream) return true;
    const double push_us = 18.0 * params / 5e6, conv_us = conv_flops / 5e8;
    return (8 * conv_us >= push_us || params * 10 > ((size_t)320 << 20)) && (!others || batch > 64);
}

// Which layers it takes: 16-bit data, a K that fits the registers, a tile for every CU (with fewer the small products' kernel and the general one put more
// workgroups on the chip), offsets within a tile in 31 bits.  Not with the sum of a replica's gradients, a third array read and written: nothing
// runs beside the local steps of a replica, and a CU's four waves are not enough for it (4096 x 9216, 32 images 177 us in gemm_kernel, 190 here).
bool fc_push_applies(int dtype, int M, int N, int K, const Epilogue &ep)
{
    return dtype == kBF16 && ep.upd_w && ep.upd_slim && !ep.upd_acc && K >= 1 && K <= 256 && N % 8 == 0 && ep.ld % 8 == 0 && ep.ld < (1L << 22) &&
           ((M + kPushBM - 1) / kPushBM) * (long)((N + kPushBN - 1) / kPushBN) >= 256;
}

int fc_push(const void *at, long lda, int M, const void *bt, long ldb, int N, int K, const Epilogue &ep, hipStream_t s)
{
    const size_t abytes = ((size_t)(K - 1) * lda + M) * 2, bbytes = ((size_t)(K - 1) * ldb + N) * 2;
    const long tiles_m = (M + kPushBM - 1) / kPushBM, total = tiles_m * ((N + kPushBN - 1) / kPushBN);
    if (abytes > kMaxOperandBytes || bbytes > kMaxOperandBytes || total > 0x7fffffffL / 2) return -1;
    FcPush p;
    p.a = Operand{at, (unsigned)abytes}; p.b = Operand{bt, (unsigned)bbytes};
    p.lda = (unsigned)(lda * 2); p.ldb = (unsigned)(ldb * 2);
    p.M = M; p.N = N; p.K = K; p.tiles_m = (int)tiles_m; p.total = (int)total; p.ld = (unsigned)ep.ld;
    p.w = ep.upd_w; p.v = ep.upd_v; p.out = static_cast<float *>(ep.out);
    for (int c = 0; c < kPushCopies; ++c) p.copy[c] = static_cast<bf16_t *>(ep.upd_copy[c]);
    p.copies = ep.upd_copies;
    p.lr = ep.upd_lr; p.mu = ep.upd_mu; p.wd = ep.upd_wd;
    const unsigned grid = (unsigned)std::min<long>(256, total);
    const auto go = [&](auto kf) {
        constexpr int KF = decltype(kf)::value;
        hipLaunchKernelGGL((fc_push_kernel<KF, KF == 16 ? 2 : 4>), dim3(grid), dim3(256), 0, s, p);
    };
    if (K <= 32) go(std::integral_constant<int, 2>{});
    else if (K <= 64) go(std::integral_constant<int, 4>{});
    else if (K <= 128) go(std::integral_constant<int, 8>{});
    else go(std::integral_constant<int, 16>{});
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace asgd
