// Fully-connected forward passes and data gradients of up to 64 images in 16-bit data whose K is split: partial sums ws[split][M][N] of A[M][K]
// (activations or output gradients, K contiguous) times the weights, stored [N][K] or (TRANS) [K][N].
//
// What bounds it is reading the weights once (75 MB of 4096 x 9216 in 11.2 us at 6.7 TB/s with 64 KB a CU on their way, 13.5 us with 32 KB), so four K
// tiles are on their way and only as many rows as there are images are staged and multiplied.  One pass, general engine / here, us: 1024, 1024 and
// 10 outputs over 2048 inputs, 64 images 111 / 106; 4096, 4096 and 1000 over 2048, 16 to 64 images 257 to 271 / 250 to 262; the same over 9248 203 / 196
// at 32; AlexNet-style net, 32 images, gradient and its accumulation 680 / 672.  Up to 64 rows: with 128 images the multiplication takes
// longer than the loads (forward 28 / 25.7, 17 / 19.6, data gradients 20.6 / 26, 13 / 16.4).
#include <hip/hip_runtime.h>

#include "asgd_internal.h"
#include "mfma_common.h"

namespace asgd {

namespace {

constexpr int kFcBN = 128, kFcThreads = 512, kFcDepth = 4;   // columns of a tile; K tiles (of 64) on their way

struct FcSplit {
    Operand a, b;
    unsigned lda, ldb;                        // bytes from one row (TRANS: K line) to the next
    int M, N, K, b_rows, per, tiles_n;
    float *ws;
};

__device__ __forceinline__ void fc_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace

// MB: blocks of 32 rows (1 or 2).  Four waves side by side own 32 columns of 32 rows each, four more the other rows (MB = 1: they only fetch).
template <int MB, bool TRANS, bool STREAM>
__global__ __launch_bounds__(kFcThreads, 2) void fc_split_kernel(FcSplit p)
{
    using T = bf16_t;
    constexpr int D = kFcDepth, WB = TRANS ? TransTile<T, kFcBN>::BYTES : kFcBN * 128, XB = 64 * 128;
    __shared__ uint4 smem[2 * (WB + XB) / 16];
    char *sw = reinterpret_cast<char *>(smem), *sx = sw + 2 * WB;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int bid;
    {
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = blockIdx.x & 7;
        bid = x * q + (x < r ? x : r) + (blockIdx.x >> 3);
    }
    const int split = bid / p.tiles_n, tn = bid - split * p.tiles_n;
    const int kt0 = split * p.per, kend = min(p.K, (kt0 + p.per) * 64);
    const int nt = (kend - kt0 * 64 + 63) / 64;   // K tiles of this workgroup (>= 1)

    // ---- fetching: pieces of 16 bytes, tile by tile; past the end zeros
    const __amdgpu_buffer_rsrc_t ra = p.a.rsrc(), rb = p.b.rsrc();
    const int row = tid >> 3, slot = tid & 7;             // rows of K: row + 64 s, elements 8 slot ..
    const int line = tid >> 4, cc = tid & 15;             // TRANS: K lines line + 32 s, columns 8 cc ..
    int k = kt0 * 64;                                     // first K of the next tile
    const unsigned xoff = row < p.M ? (unsigned)row * p.lda : kInv;
    unsigned woff[2];
    static_for<0, 2>([&](auto s) ASGD_INLINE {
        const int n = tn * kFcBN + (TRANS ? cc * 8 : row + s * 64);
        woff[s] = n < p.b_rows ? TRANS ? (unsigned)n * 2u : (unsigned)n * p.ldb : kInv;
    });
    uint4 r[D][3];
    auto load = [&](auto set) ASGD_INLINE {
        const unsigned kc = k + slot * 8 < kend ? (unsigned)(k + slot * 8) * 2u : kInv;
        static_for<0, 2>([&](auto s) ASGD_INLINE {
            const int kl = k + line + s * 32;
            r[set][s] = buf_ld16<STREAM>(rb, woff[s] + (TRANS ? (kl < kend ? (unsigned)kl * p.ldb : kInv) : kc));
        });
        r[set][2] = buf_ld16(ra, xoff + kc);
        k += 64;
    };
    const unsigned so = (unsigned)(row * 8 + (slot ^ swz(row))) * 16u;   // rows 64 apart share the swizzle
    auto store = [&](auto set, auto buf) ASGD_INLINE {
        static_for<0, 2>([&](auto s) ASGD_INLINE {
            const unsigned o = TRANS ? (unsigned)((line + s * 32) * TransTile<T, kFcBN>::LINE + cc * 16) : so + s * (64 * 128);
            *reinterpret_cast<uint4 *>(sw + buf * WB + o) = r[set][s];
        });
        *reinterpret_cast<uint4 *>(sx + buf * XB + so) = r[set][2];
    };

    // ---- multiplying
    const int n0 = (wave & 3) * 32, m0 = (wave >> 2) * 32;
    const bool busy = m0 < 32 * MB && m0 < p.M && tn * kFcBN + n0 < p.N;   // wave-uniform
    FragOff<T, TRANS, kFcBN> fow;
    FragOff<T, false, 64> fox;
    fow.init(n0, lane);
    fox.init(m0, lane);
    f32x16 acc = {};
    auto multiply = [&](auto buf) ASGD_INLINE {
        const char *w = sw + buf * WB, *x = sx + buf * XB;
        Frag<T> fw[2], fx[2];
        fw[0].template read<0, 0>(w, fow);
        fx[0].template read<0, 0>(x, fox);
        static_for<0, 4>([&](auto ks) ASGD_INLINE {
            constexpr int cur = ks % 2, nxt = (ks + 1) % 2;
            if constexpr (ks < 3) {
                fw[nxt].template read<ks + 1, 0>(w, fow);
                fx[nxt].template read<ks + 1, 0>(x, fox);
            }
            mma(acc, fx[cur], fw[cur]);
        });
    };
    static_for<0, D>([&](auto d) ASGD_INLINE { load(d); });
    store(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
    load(std::integral_constant<int, 0>{});
    // Whole rounds of four steps without a condition, so that the compiler's wait counts are exact: a step waits for the loads of four steps ago.
    // Past the last tile zeros are fetched and added.
    for (int t = 0; t < nt; t += 4) {
        static_for<0, 4>([&](auto u) ASGD_INLINE {
            constexpr int set = (u + 1) % D;
            fc_barrier();
            if (busy) multiply(std::integral_constant<int, u % 2>{});
            store(std::integral_constant<int, set>{}, std::integral_constant<int, (u + 1) % 2>{});
            load(std::integral_constant<int, set>{});
        });
    }
    // ---- partial sums: a lane has one column of 16 rows, a store instruction two whole lines
    if (!busy) return;
    const int n = tn * kFcBN + n0 + (lane & 31), half = lane >> 5;
    if (n >= p.N) return;
    static_for<0, 16>([&](auto v) ASGD_INLINE {
        const int m = m0 + 8 * (v / 4) + 4 * half + v % 4;
        if (m < p.M) p.ws[((size_t)split * p.M + m) * p.N + n] = acc[decltype(v)::value];
    });
}

// Weights that stay in the memory-side cache (256 MB) from one pass to the next are read by ordinary loads.  Where what a pass writes between two uses
// pushes them out they are non-temporal: on its way through the caches an ordinary load then pushes out what the kernels before have written, and
// waits for it (4096 outputs over 9216 inputs inside a pass of 32 images 28.0 us, non-temporal 16.9).  Ordinary / non-temporal: 4096, 4096
// and 1000 outputs over 9248 inputs, 64 images, gradient 207 / 227 us, step 379 / 403; AlexNet-style step in calls, 16 images 664 / 679, 32 759 / 760; gradient
// and accumulation, 32 images 678 / 672, 48 803 / 787; replays of 2 x 16 images 4768 / 4722, 4 x 16 4870 / 4820, 4 x 32 5594 / 5595; 13 M parameters
// behind a small convolution, replay of 4 x 48 images 1041 / 1076, 59 M 3125 / 3174.  (Against the rule: 59 M, gradient and accumulation, 340 / 327; 34 M, replay
// of 2 x 48 images 1793 / 1727.)
bool fc_split_streams(size_t weights, size_t workspace, int replicas) { return weights + workspace * replicas > ((size_t)256 << 20); }

int fc_split(bool trans, const void *a, long lda, int M, const void *b, long ldb, int N, int b_rows, int K, int splits, bool stream, float *ws, hipStream_t s)
{
    FcSplit p;
    const size_t ab = ((size_t)(M - 1) * lda + K) * 2, bb = trans ? ((size_t)(K - 1) * ldb + N) * 2 : ((size_t)(b_rows - 1) * ldb + K) * 2;
    if (M > 64 || ab > kMaxOperandBytes || bb > kMaxOperandBytes || !ws) return -1;
    p.a = Operand{a, (unsigned)ab}; p.b = Operand{b, (unsigned)bb};
    p.lda = (unsigned)(lda * 2); p.ldb = (unsigned)(ldb * 2);
    p.M = M; p.N = N; p.K = K; p.b_rows = trans ? N : b_rows;
    const int nkt = (K + 63) / 64;
    p.per = (nkt + splits - 1) / splits;
    p.tiles_n = (N + kFcBN - 1) / kFcBN; p.ws = ws;
    const long grid = (long)p.tiles_n * splits;
    if (grid <= 0 || grid > 0x7fffffffL || (long)(splits - 1) * p.per >= nkt) return -1;
    const auto go = [&](auto m, auto t) {
        constexpr int MB = decltype(m)::value;
        constexpr bool TRANS = decltype(t)::value;
        if (stream) hipLaunchKernelGGL((fc_split_kernel<MB, TRANS, true>), dim3((unsigned)grid), dim3(kFcThreads), 0, s, p);
        else hipLaunchKernelGGL((fc_split_kernel<MB, TRANS, false>), dim3((unsigned)grid), dim3(kFcThreads), 0, s, p);
    };
    const auto rows = [&](auto t) {
        if (M <= 32) go(std::integral_constant<int, 1>{}, t);
        else go(std::integral_constant<int, 2>{}, t);
    };
    if (trans) rows(std::true_type{});
    else rows(std::false_type{});
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace asgd
