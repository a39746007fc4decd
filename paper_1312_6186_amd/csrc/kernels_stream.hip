// Bandwidth-bound kernels of the hot path for gfx950: the fused momentum /
// weight-decay update (optionally writing the worker copy in the same pass), the
// Adagrad / Adadelta updates, the gradient accumulator, the parameter snapshot,
// pooling, response normalisation, softmax cross-entropy, bias-gradient column
// sums and the layout conversions around the channel-last activation format.
// Every reduction has a fixed summation order so that a run is reproducible bit
// for bit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "asgd_internal.h"
#include "mfma_common.h"
#include "reduce.h"

namespace asgd {

__device__ inline float ldf(const float *p) { return *p; }
__device__ inline float ldf(const bf16_t *p) { return (float)*p; }
__device__ inline void stf(float *p, float v) { *p = v; }
__device__ inline void stf(bf16_t *p, float v) { *p = (bf16_t)v; }

static inline unsigned blocks_for(size_t n, unsigned per_block) { return (unsigned)((n + per_block - 1) / per_block); }
static inline int launch_ok() { return hipGetLastError() == hipSuccess ? 0 : -1; }

uint64_t dropout_key(uint64_t seed, uint64_t step, uint32_t worker, uint32_t layer)
{
    return mix64(mix64(mix64(seed) + step) + (((uint64_t)worker << 32) | (uint64_t)layer));
}

// ---------------------------------------------------------------- update
// t = g + wd*w; v = mu*v - lr*t; w = w + v.  20 bytes of traffic per parameter.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Each thread owns 4 float4 per buffer, 256 apart, all loads issued before the arithmetic; gradients are read and
// parameters / momentum written with non-temporal hints (the 1.2 GB working set of the AlexNet-style net cannot
// stay in cache between steps anyway).  Measured 5.65 TB/s on 62.4 M parameters.
// One element of the update, with the contractions written out so that every code path (vector body, scalar
// tail, unaligned fallback) rounds identically: t = g + wd*w;  v = mu*v - lr*t;  w = w + v.
__device__ __forceinline__ void update1(float &w, float &v, float g, float lr, float mu, float wd)
{
    const float t = __builtin_fmaf(wd, w, g);
    v = __builtin_fmaf(mu, v, -(lr * t));
    w = w + v;
}

template <bool ONCE> __device__ __forceinline__ f32x4 load4(const f32x4 *p)
{
    if constexpr (ONCE) return __builtin_nontemporal_load(p);
    else return *p;
}

// SNAP: 0 = update only, 1 = also write the new parameters to `copy` as fp32, 2 = as bf16 (round to nearest even):
// the worker copy of the next fetch comes out of the same pass instead of a second read of the parameters.
__device__ inline uint32_t f32_to_bf16_bits(uint32_t u);
// The work of block `blk` of an update over n parameters whose buffers are 16-byte aligned (n4 = n / 4 whole vectors;
// block 0 also takes the n % 4 elements behind them).
template <int SNAP, bool ONCE>
__device__ __forceinline__ void update_block(f32x4 *__restrict__ w, f32x4 *__restrict__ v, const f32x4 *__restrict__ g, size_t n4, float *ws, float *vs,
                                             const float *gs, size_t n, float lr, float mu, float wd, void *__restrict__ copy, size_t blk)
{
    constexpr int U = 4;
    const size_t i0 = blk * (256 * U) + threadIdx.x;
    f32x4 ww[U], vv[U], gg[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t i = i0 + (size_t)u * 256;
        if (i < n4) { ww[u] = load4<ONCE>(&w[i]); vv[u] = load4<ONCE>(&v[i]); gg[u] = __builtin_nontemporal_load(&g[i]); }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t i = i0 + (size_t)u * 256;
        if (i < n4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float wn = ww[u][e], vn = vv[u][e];
                update1(wn, vn, gg[u][e], lr, mu, wd);
                ww[u][e] = wn; vv[u][e] = vn;
            }
            __builtin_nontemporal_store(ww[u], &w[i]);
            __builtin_nontemporal_store(vv[u], &v[i]);
            if constexpr (SNAP == 1) static_cast<f32x4 *>(copy)[i] = ww[u];
            if constexpr (SNAP == 2) {
                typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
                u32x2 o;
                o.x = f32_to_bf16_bits(__float_as_uint(ww[u].x)) | (f32_to_bf16_bits(__float_as_uint(ww[u].y)) << 16);
                o.y = f32_to_bf16_bits(__float_as_uint(ww[u].z)) | (f32_to_bf16_bits(__float_as_uint(ww[u].w)) << 16);
                static_cast<u32x2 *>(copy)[i] = o;
            }
        }
    }
    if (blk == 0) {
        const size_t i = n4 * 4 + threadIdx.x;
        if (i < n) {
            float wn = ws[i], vn = vs[i];
            update1(wn, vn, gs[i], lr, mu, wd);
            vs[i] = vn; ws[i] = wn;
            if constexpr (SNAP == 1) static_cast<float *>(copy)[i] = wn;
            if constexpr (SNAP == 2) static_cast<uint16_t *>(copy)[i] = (uint16_t)f32_to_bf16_bits(__float_as_uint(wn));
        }
    }
}

template <int SNAP, bool ONCE>
__global__ __launch_bounds__(256) void update_kernel(f32x4 *__restrict__ w, f32x4 *__restrict__ v, const f32x4 *__restrict__ g, size_t n4,
                                                     float *ws, float *vs, const float *gs, size_t n, float lr, float mu, float wd,
                                                     int *version_counter, void *__restrict__ copy)
{
    update_block<SNAP, ONCE>(w, v, g, n4, ws, vs, gs, n, lr, mu, wd, copy, blockIdx.x);
    if (blockIdx.x == 0 && threadIdx.x == 0 && version_counter) *version_counter += 1;
}

// The same over up to eight separate ranges of one parameter vector in one launch, with a replay's accumulator, copies and log in
// the same pass (PushRanges): a block finds its range.  A range whose start is not a multiple of 4 elements runs element by
// element.  Bound by memory.  62.4 M parameters: 204 us without a copy (the update 209, each fetch by a snapshot of its own 75 more); 2
// bytes more a parameter and copy in bf16.
__device__ __forceinline__ uint2 bf16x4(const f32x4 &v)
{
    return make_uint2(f32_to_bf16_bits(__float_as_uint(v.x)) | (f32_to_bf16_bits(__float_as_uint(v.y)) << 16),
                      f32_to_bf16_bits(__float_as_uint(v.z)) | (f32_to_bf16_bits(__float_as_uint(v.w)) << 16));
}
__device__ __forceinline__ void push_one(const PushRanges &p, size_t i)
{
    const float g = p.g[i];
    float wn = p.w[i], vn = p.v[i];
    update1(wn, vn, g, p.lr, p.mu, p.wd);
    if (p.acc) p.acc[i] = p.acc_first ? g : p.acc[i] + g;
    p.v[i] = vn; p.w[i] = wn;
    for (int c = 0; c < p.ncopies; ++c) {
        if (p.f32mask >> c & 1) static_cast<float *>(p.copy[c])[i] = wn;
        else static_cast<uint16_t *>(p.copy[c])[i] = (uint16_t)f32_to_bf16_bits(__float_as_uint(wn));
    }
}
__global__ __launch_bounds__(256) void push_ranges_kernel(PushRanges p)
{
    int q = 0;
    while (q + 1 < p.n && blockIdx.x >= p.blk[q + 1]) ++q;
    const size_t off = p.off[q], n = p.cnt[q], blk = blockIdx.x - p.blk[q];
    if (blockIdx.x == 0 && threadIdx.x == 0 && p.counter) {
        const int version = *p.counter + 1;
        *p.counter = version;
        for (int c = 0; c < p.nlogs; ++c) { p.log[c][0] = p.log_update[c]; p.log[c][1] = p.log_worker[c]; p.log[c][2] = version; }
    }
    if ((off & 3) != 0) {
        for (size_t i = blk * 1024 + threadIdx.x; i < n && i < (blk + 1) * 1024; i += 256) push_one(p, off + i);
        return;
    }
    constexpr int U = 4;
    const size_t n4 = n / 4, i0 = blk * (256 * U) + threadIdx.x;
    f32x4 *w = reinterpret_cast<f32x4 *>(p.w + off), *v = reinterpret_cast<f32x4 *>(p.v + off), *acc = reinterpret_cast<f32x4 *>(p.acc ? p.acc + off : nullptr);
    const f32x4 *g = reinterpret_cast<const f32x4 *>(p.g + off);
    const bool add = p.acc && !p.acc_first;
    f32x4 ww[U], vv[U], gg[U], aa[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t i = i0 + (size_t)u * 256;
        if (i < n4) {
            ww[u] = w[i]; vv[u] = v[i]; gg[u] = __builtin_nontemporal_load(&g[i]);
            if (add) aa[u] = __builtin_nontemporal_load(&acc[i]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t i = i0 + (size_t)u * 256;
        if (i >= n4) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float wn = ww[u][e], vn = vv[u][e];
            update1(wn, vn, gg[u][e], p.lr, p.mu, p.wd);
            ww[u][e] = wn; vv[u][e] = vn;
            if (add) gg[u][e] = aa[u][e] + gg[u][e];
        }
        __builtin_nontemporal_store(ww[u], &w[i]);
        __builtin_nontemporal_store(vv[u], &v[i]);
        if (p.acc) __builtin_nontemporal_store(gg[u], &acc[i]);
        for (int c = 0; c < p.ncopies; ++c) {
            if (p.f32mask >> c & 1) reinterpret_cast<f32x4 *>(static_cast<float *>(p.copy[c]) + off)[i] = ww[u];
            else reinterpret_cast<uint2 *>(static_cast<uint16_t *>(p.copy[c]) + off)[i] = bf16x4(ww[u]);
        }
    }
    if (blk == 0 && n4 * 4 + threadIdx.x < n) push_one(p, off + n4 * 4 + threadIdx.x);
}

template <int SNAP>
__global__ __launch_bounds__(256) void update_scalar_kernel(float *w, float *v, const float *g, size_t n, float lr, float mu, float wd,
                                                            int *version_counter, void *copy)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        float wn = w[i], vn = v[i];
        update1(wn, vn, g[i], lr, mu, wd);
        v[i] = vn; w[i] = wn;
        if constexpr (SNAP == 1) static_cast<float *>(copy)[i] = wn;
        if constexpr (SNAP == 2) static_cast<uint16_t *>(copy)[i] = (uint16_t)f32_to_bf16_bits(__float_as_uint(wn));
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && version_counter) *version_counter += 1;
}

bool beyond_cache(size_t n, int arrays, size_t copy_es) { return n * (4 * (size_t)arrays + copy_es) > ((size_t)384 << 20); }

template <int SNAP>
static int launch_update_t(float *w, float *v, const float *g, size_t n, size_t total, float lr, float mu, float wd, int *version_counter, void *copy, hipStream_t s)
{
    const unsigned copy_align = SNAP == 1 ? 15u : SNAP == 2 ? 7u : 0u;
    const bool aligned = (((uintptr_t)w | (uintptr_t)v | (uintptr_t)g) & 15) == 0 && ((uintptr_t)copy & copy_align) == 0;
    if (aligned && n >= 4) {
        const size_t n4 = n / 4;
        const size_t blocks = (n4 + 1023) / 1024 ? (n4 + 1023) / 1024 : 1;
        if (blocks > 0x7fffffffu) return -1;
        const auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, reinterpret_cast<f32x4 *>(w), reinterpret_cast<f32x4 *>(v),
                               reinterpret_cast<const f32x4 *>(g), n4, w, v, g, n, lr, mu, wd, version_counter, copy);
        };
        if (beyond_cache(total, 2, SNAP == 1 ? 4 : SNAP == 2 ? 2 : 0)) go(update_kernel<SNAP, true>);
        else go(update_kernel<SNAP, false>);
    } else {
        unsigned blocks = blocks_for(n ? n : 1, 256);
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL(update_scalar_kernel<SNAP>, dim3(blocks), dim3(256), 0, s, w, v, g, n, lr, mu, wd, version_counter, copy);
    }
    return launch_ok();
}
int launch_update(float *w, float *v, const float *g, size_t n, float lr, float mu, float wd, int *version_counter, hipStream_t s)
{
    return launch_update_t<0>(w, v, g, n, n, lr, mu, wd, version_counter, nullptr, s);
}
int launch_push_ranges(PushRanges &p, hipStream_t s)
{
    if (p.n <= 0) return 0;
    if (p.n > 8 || p.ncopies > 2 * kPushCopies || p.nlogs > kPushCopies) return -1;
    uintptr_t align = (uintptr_t)p.w | (uintptr_t)p.v | (uintptr_t)p.g | (uintptr_t)p.acc;
    for (int c = 0; c < p.ncopies; ++c) align |= (uintptr_t)p.copy[c];
    if (align & 15) return -1;
    size_t blocks = 0;
    for (int q = 0; q < p.n; ++q) {
        p.blk[q] = (unsigned)blocks;
        const size_t b = (p.off[q] & 3) == 0 ? (p.cnt[q] / 4 + 1023) / 1024 : (p.cnt[q] + 1023) / 1024;   // 1024 vectors, or 1024 elements, per block
        blocks += b ? b : 1;
        if (blocks > 0x7fffffffu) return -1;
    }
    p.blk[p.n] = (unsigned)blocks;
    hipLaunchKernelGGL(push_ranges_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p);
    return launch_ok();
}
int launch_update_snapshot(float *w, float *v, const float *g, size_t n, size_t total, float lr, float mu, float wd, void *copy, int dst_dtype, hipStream_t s)
{
    if (dst_dtype == kBF16) return launch_update_t<2>(w, v, g, n, total, lr, mu, wd, nullptr, copy, s);
    return launch_update_t<1>(w, v, g, n, total, lr, mu, wd, nullptr, copy, s);
}

// ---------------------------------------------------------------- Adagrad / Adadelta server updates
// The same streaming shape as the momentum update: 16-byte vectors where the buffers allow, identical arithmetic
// (explicit contractions) on every path.
//   Adagrad :  t = g + wd*w;  h += t*t;  w -= lr * t / (sqrt(h) + eps)
//   Adadelta:  t = g + wd*w;  a = rho*a + (1-rho)*t*t;  d = -sqrt(b+eps)/sqrt(a+eps)*t;  b = rho*b + (1-rho)*d*d;  w += d
__device__ __forceinline__ void adagrad1(float &w, float &h, float g, float lr, float eps, float wd)
{
    const float t = __builtin_fmaf(wd, w, g);
    h = __builtin_fmaf(t, t, h);
    w = w - lr * t * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(h) + eps);   // hardware sqrt and reciprocal: about an ulp each on the step
}
__device__ __forceinline__ void adadelta1(float &w, float &a, float &b, float g, float rho, float eps, float wd)
{
    const float t = __builtin_fmaf(wd, w, g);
    a = __builtin_fmaf(rho, a, (1.f - rho) * (t * t));
    const float d = -(__builtin_amdgcn_sqrtf(b + eps) * __builtin_amdgcn_rsqf(a + eps)) * t;   // hardware sqrt and reciprocal sqrt
    b = __builtin_fmaf(rho, b, (1.f - rho) * (d * d));
    w = w + d;
}
// KIND 0: Adagrad (s1 = h, s2 unused, c1 = lr); KIND 1: Adadelta (s1 = a, s2 = b, c1 = rho)
template <int KIND, bool ONCE>
__global__ __launch_bounds__(256) void adaptive_update_kernel(float *__restrict__ w, float *__restrict__ s1, float *__restrict__ s2,
                                                             const float *__restrict__ g, size_t n, int vec, float c1, float eps, float wd)
{
    // vector body: each thread owns U float4 per buffer, 256 apart, all loads issued before the arithmetic
    constexpr int U = 4;
    const size_t n4 = vec ? n / 4 : 0;
    const size_t i0 = (size_t)blockIdx.x * (256 * U) + threadIdx.x;
    f32x4 ww[U], aa[U], bb[U], gg[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t i = i0 + (size_t)u * 256;
        if (i < n4) {
            ww[u] = load4<ONCE>(&reinterpret_cast<f32x4 *>(w)[i]); aa[u] = load4<ONCE>(&reinterpret_cast<f32x4 *>(s1)[i]);
            if (KIND == 1) bb[u] = load4<ONCE>(&reinterpret_cast<f32x4 *>(s2)[i]);
            gg[u] = __builtin_nontemporal_load(&reinterpret_cast<const f32x4 *>(g)[i]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t i = i0 + (size_t)u * 256;
        if (i < n4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float we = ww[u][e], ae = aa[u][e], be = KIND == 1 ? bb[u][e] : 0.f;
                if (KIND == 0) adagrad1(we, ae, gg[u][e], c1, eps, wd);
                else adadelta1(we, ae, be, gg[u][e], c1, eps, wd);
                ww[u][e] = we; aa[u][e] = ae;
                if (KIND == 1) bb[u][e] = be;
            }
            __builtin_nontemporal_store(ww[u], &reinterpret_cast<f32x4 *>(w)[i]);
            __builtin_nontemporal_store(aa[u], &reinterpret_cast<f32x4 *>(s1)[i]);
            if (KIND == 1) __builtin_nontemporal_store(bb[u], &reinterpret_cast<f32x4 *>(s2)[i]);
        }
    }
    // scalar tail (everything, if the buffers are not 16-byte aligned), grid-stride
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = n4 * 4 + (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        float we = w[i], ae = s1[i], be = KIND == 1 ? s2[i] : 0.f;
        if (KIND == 0) adagrad1(we, ae, g[i], c1, eps, wd);
        else adadelta1(we, ae, be, g[i], c1, eps, wd);
        w[i] = we; s1[i] = ae;
        if (KIND == 1) s2[i] = be;
    }
}
static unsigned adaptive_blocks(size_t n, int vec)
{
    if (vec) { const size_t b = (n / 4 + 1023) / 1024; return (unsigned)(b ? b : 1); }
    unsigned b = blocks_for(n ? n : 1, 256);
    return b > 32768 ? 32768 : b;
}
int launch_adagrad(float *w, float *h, const float *g, size_t n, float lr, float eps, float wd, hipStream_t s)
{
    const int vec = ((((uintptr_t)w | (uintptr_t)h | (uintptr_t)g) & 15) == 0) ? 1 : 0;
    const unsigned blocks = adaptive_blocks(n, vec);
    const auto kernel = beyond_cache(n, 2, 0) ? adaptive_update_kernel<0, true> : adaptive_update_kernel<0, false>;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, w, h, static_cast<float *>(nullptr), g, n, vec, lr, eps, wd);
    return launch_ok();
}
int launch_adadelta(float *w, float *a, float *b, const float *g, size_t n, float rho, float eps, float wd, hipStream_t s)
{
    const int vec = ((((uintptr_t)w | (uintptr_t)a | (uintptr_t)b | (uintptr_t)g) & 15) == 0) ? 1 : 0;
    const unsigned blocks = adaptive_blocks(n, vec);
    const auto kernel = beyond_cache(n, 3, 0) ? adaptive_update_kernel<1, true> : adaptive_update_kernel<1, false>;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, w, a, b, g, n, vec, rho, eps, wd);
    return launch_ok();
}

// ---------------------------------------------------------------- gradient accumulator (n_push > 1)
// acc = g (first) or acc + g; 16-byte vectors when both are aligned, the same arithmetic either way.
__global__ __launch_bounds__(256) void accumulate_kernel(float *__restrict__ acc, const float *__restrict__ g, size_t n, int first, int vec)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t n4 = vec ? n / 4 : 0;
    for (size_t i = t0; i < n4; i += stride) {
        f32x4 a = __builtin_nontemporal_load(&reinterpret_cast<const f32x4 *>(g)[i]);
        if (!first) a += reinterpret_cast<f32x4 *>(acc)[i];
        reinterpret_cast<f32x4 *>(acc)[i] = a;
    }
    for (size_t i = n4 * 4 + t0; i < n; i += stride) acc[i] = first ? g[i] : acc[i] + g[i];
}
int launch_accumulate(float *acc, const float *g, size_t n, bool first, hipStream_t s)
{
    const int vec = ((((uintptr_t)acc | (uintptr_t)g) & 15) == 0) ? 1 : 0;
    unsigned blocks = blocks_for(vec ? (n + 3) / 4 : n, 256);
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(accumulate_kernel, dim3(blocks), dim3(256), 0, s, acc, g, n, first ? 1 : 0, vec);
    return launch_ok();
}

// ---------------------------------------------------------------- snapshot
__device__ inline uint32_t f32_to_bf16_bits(uint32_t u)  // round to nearest even; NaN -> quiet NaN
{
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (u >> 16) | 0x0040u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__global__ __launch_bounds__(256) void snapshot_kernel(const float *__restrict__ src, void *__restrict__ dst, size_t n, int to_bf16, int vec,
                                                       const int *version_counter, int32_t *log_slot, int log_update, int log_worker)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t0 == 0 && log_slot) {
        log_slot[0] = log_update;
        log_slot[1] = log_worker;
        log_slot[2] = version_counter ? *version_counter : -1;
    }
    if (!to_bf16) {
        float *d = static_cast<float *>(dst);
        const size_t n4 = vec ? n / 4 : 0;
        for (size_t i = t0; i < n4; i += stride) reinterpret_cast<float4 *>(d)[i] = reinterpret_cast<const float4 *>(src)[i];
        for (size_t i = n4 * 4 + t0; i < n; i += stride) d[i] = src[i];
    } else {
        uint16_t *d = static_cast<uint16_t *>(dst);
        const size_t n8 = vec ? n / 8 : 0;
        // groups of 8 elements; a thread takes four of them per round, 256 apart, and issues its eight loads first
        typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
        constexpr int U = 4;
        for (size_t base = (size_t)blockIdx.x * (256 * U); base < n8; base += (size_t)gridDim.x * (256 * U)) {
            u32x4v a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t i = base + threadIdx.x + (size_t)u * 256;
                if (i < n8) {
                    a[u] = __builtin_nontemporal_load(&reinterpret_cast<const u32x4v *>(src)[2 * i]);
                    b[u] = __builtin_nontemporal_load(&reinterpret_cast<const u32x4v *>(src)[2 * i + 1]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t i = base + threadIdx.x + (size_t)u * 256;
                if (i < n8) {
                    uint4 o;
                    o.x = f32_to_bf16_bits(a[u].x) | (f32_to_bf16_bits(a[u].y) << 16);
                    o.y = f32_to_bf16_bits(a[u].z) | (f32_to_bf16_bits(a[u].w) << 16);
                    o.z = f32_to_bf16_bits(b[u].x) | (f32_to_bf16_bits(b[u].y) << 16);
                    o.w = f32_to_bf16_bits(b[u].z) | (f32_to_bf16_bits(b[u].w) << 16);
                    reinterpret_cast<uint4 *>(d)[i] = o;
                }
            }
        }
        for (size_t i = n8 * 8 + t0; i < n; i += stride) d[i] = (uint16_t)f32_to_bf16_bits(__float_as_uint(src[i]));
    }
}

int launch_snapshot(const float *src, void *dst, size_t n, int dst_dtype, const int *version_counter, int32_t *log_slot, int log_update,
                    int log_worker, hipStream_t s)
{
    const int vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    const size_t per = dst_dtype == kBF16 ? 8 : 4;
    unsigned blocks = blocks_for(n / per + 1, 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(snapshot_kernel, dim3(blocks), dim3(256), 0, s, src, dst, n, dst_dtype == kBF16 ? 1 : 0, vec, version_counter, log_slot,
                       log_update, log_worker);
    return launch_ok();
}

// ---------------------------------------------------------------- fill
__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t *p, size_t words)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) p[i] = 0u;
}
int launch_fill_zero(void *p, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return 0;
    if ((bytes & 3) || ((uintptr_t)p & 3)) return -1;
    unsigned blocks = blocks_for(bytes / 4, 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, static_cast<uint32_t *>(p), bytes / 4);
    return launch_ok();
}

// ---------------------------------------------------------------- input staging and filter packing
__device__ __forceinline__ uint32_t fdiv32(uint32_t n, const FastDiv &f) { return (__umulhi(n, f.mul) + n) >> f.sh; }
// One element of work of the input staging: images [B][C][H][W] -> the first layer's channel-last input.
// FORM 0: 16 bytes of channels of one pixel, Cp channels per pixel, zeros past C (reads contiguous along w for each channel).
// FORM 1..4: FORM channels per pixel into the interior of a bordered tensor, PX neighbouring pixels of one row.  PX = 4 (W and
// the image base allow 4-element loads): one load per channel; PX = 2 (even W): element loads; PX = 1: any width, element
// stores.  For PX > 1 the elements make a whole number of dwords at a dword-aligned address (checked by the launcher).
template <typename T, int FORM, int PX> __device__ __forceinline__ void stage_one(const StageJob &j, unsigned i)
{
    const T *__restrict__ src = static_cast<const T *>(j.src);
    T *__restrict__ dst = static_cast<T *>(j.dst);
    if constexpr (FORM == 0) {
        constexpr int V = 16 / sizeof(T);
        const unsigned per = (unsigned)j.B * j.H * j.W, gidx = i / per, pix = i - gidx * per;   // pixels fastest
        const unsigned n = fdiv32(pix, j.dHW), hw = pix - n * (unsigned)(j.H * j.W);
        union { uint4 u; T e[V]; } v;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int c = (int)gidx * V + e;
            v.e[e] = c < j.C ? src[((size_t)n * j.C + c) * (size_t)(j.H * j.W) + hw] : (T)0.f;
        }
        *reinterpret_cast<uint4 *>(dst + (size_t)pix * j.Cp + gidx * V) = v.u;
    } else {
        constexpr int PC = FORM;
        const size_t HW = (size_t)j.H * j.W;
        const unsigned row = fdiv32(i, j.dWq), w = (i - row * j.dWq.d) * PX;     // row = n * H + h
        const unsigned n = fdiv32(row, j.dH), h = row - n * (unsigned)j.H;
        const T *s0 = src + (size_t)n * j.C * HW + (size_t)h * j.W + w;
        union { T e[PX * PC]; uint32_t u[(PX * PC * sizeof(T) + 3) / 4]; } v;
        if constexpr (PX == 4) {
            typedef T t4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int c = 0; c < PC; ++c) {
                const t4 x = c < j.C ? *reinterpret_cast<const t4 *>(s0 + c * HW) : t4{};
#pragma unroll
                for (int q = 0; q < 4; ++q) v.e[q * PC + c] = x[q];
            }
        } else {
#pragma unroll
            for (int q = 0; q < PX; ++q)
#pragma unroll
                for (int c = 0; c < PC; ++c) v.e[q * PC + c] = c < j.C ? s0[c * HW + q] : (T)0.f;
        }
        T *o = dst + (((size_t)n * (j.H + 2 * j.pad) + h + j.pad) * j.Wp + w + j.pad) * PC;
        if constexpr (PX > 1) {
            uint32_t *o4 = reinterpret_cast<uint32_t *>(o);
#pragma unroll
            for (int q = 0; q < (int)(PX * PC * sizeof(T) / 4); ++q) o4[q] = v.u[q];
        } else {
#pragma unroll
            for (int c = 0; c < PC; ++c) o[c] = v.e[c];
        }
    }
}
// Element (row n, window position pos, channel c) of a filter pack in the order of conv_direct.
__device__ __forceinline__ long direct_index(int n, int pos, int c, int ks, int nch, int npos)
{
    const int cw = ks * 16, ch = c / cw, e = c - ch * cw;
    return ((((long)(n >> 5) * nch + ch) * npos + pos) * ks + (e >> 4)) * 512 + ((n & 31) + 32 * ((e >> 3) & 1)) * 8 + (e & 7);
}
// All convolution layers of a net in one launch.  A thread produces 8 consecutive packed elements (the innermost
// packed index is a multiple of 8 wide in every pack) and stores them as one or two 16-byte vectors; group g
// belongs to the job whose range holds it.
template <typename T> __global__ __launch_bounds__(256) void pack_conv_kernel(PackJobs jobs)
{
    const unsigned g = blockIdx.x * 256u + threadIdx.x;
    if (g >= jobs.total) return;
    int q = 0;
    while (q + 1 < jobs.n && g >= jobs.j[q + 1].start) ++q;
    const PackJob &J = jobs.j[q];
    const T *w = static_cast<const T *>(J.w);
    unsigned li = (g - J.start) * 8u;     // first of this thread's 8 elements
    const int k = J.k;
    const long kk = (long)k * k;
    __attribute__((aligned(16))) T out[8];
    T *dst;
    if (J.rw) {  // wf[co][ky][j], j = kx*rw + ci over a padded window row of KW elements (rw channels per stored pixel)
        const int j0 = (int)(li % (unsigned)J.KW); unsigned t = li / (unsigned)J.KW;
        const int ky = (int)(t % (unsigned)k), co = (int)(t / (unsigned)k);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int kx = (j0 + e) / J.rw, ci = (j0 + e) - kx * J.rw;
            out[e] = (co < J.cout && ci < J.cin && kx < k) ? w[((long)co * J.cin + ci) * kk + ky * k + kx] : (T)0.f;
        }
        dst = static_cast<T *>(J.wf) + li;
    } else if (li < J.nf) {  // wf[co][ky][kx][ci], with zeros up to the end of the last chunk
        const int ci0 = (int)(li % (unsigned)J.cinw); unsigned t = li / (unsigned)J.cinw;
        const int kx = (int)(t % (unsigned)k); t /= (unsigned)k;
        const int ky = (int)(t % (unsigned)k), co = (int)(t / (unsigned)k);
        const T *src = w + ((long)co * J.cin + ci0) * kk + ky * k + kx;
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = (co < J.cout && ci0 + e < J.cin) ? src[e * kk] : (T)0.f;
        dst = static_cast<T *>(J.wf) + (J.fks ? direct_index(co, ky * k + kx, ci0, J.fks, J.fch, (int)kk) : (long)li);
    } else {  // wd[ci][ky'][kx'][co] = w[co][ci][k-1-ky'][k-1-kx']
        li -= J.nf;
        const int co0 = (int)(li % (unsigned)J.coutp); unsigned t = li / (unsigned)J.coutp;
        const int kx = (int)(t % (unsigned)k); t /= (unsigned)k;
        const int ky = (int)(t % (unsigned)k), ci = (int)(t / (unsigned)k);
        const T *src = w + ((long)co0 * J.cin + ci) * kk + (k - 1 - ky) * k + (k - 1 - kx);
        const long cstride = (long)J.cin * kk;
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = (co0 + e < J.cout && ci < J.cin) ? src[e * cstride] : (T)0.f;
        dst = static_cast<T *>(J.wd) + (J.dks ? direct_index(ci, ky * k + kx, co0, J.dks, J.dch, (int)kk) : (long)li);
    }
    uint4 *d4 = reinterpret_cast<uint4 *>(dst);
    const uint4 *o4 = reinterpret_cast<const uint4 *>(out);
#pragma unroll
    for (int v = 0; v < (int)(8 * sizeof(T) / 16); ++v) d4[v] = o4[v];
}
// The same through LDS, for layers whose filters of 16 bytes' worth of output channels (8 in bf16, 4 in fp32) fit
// into 64 KB: a workgroup owns such a group of output channels, copies its filters (one contiguous, 16-byte aligned
// run of the canonical tensor) into LDS with 16-byte loads and writes every packed vector that holds them.  The
// gather form above reads its 8 elements k*k apart, 2 or 4 bytes at a time.
template <typename T> __device__ __forceinline__ void pack_lds_block(const PackJobs &jobs, uint4 *slab4)
{
    constexpr int V = 16 / (int)sizeof(T), NT = 1024;
    T *slab = reinterpret_cast<T *>(slab4);
    int q = 0;
    while (q + 1 < jobs.n && blockIdx.x >= jobs.j[q + 1].start) ++q;
    const PackJob &J = jobs.j[q];
    const int tid = threadIdx.x;
    const int co0 = (int)(blockIdx.x - J.start) * V;
    const int k = J.k, kk = k * k, S = J.cin * kk;   // S: elements per output channel
    const long left = (long)J.cout * S - (long)co0 * S;
    const int n_el = (int)(left < (long)V * S ? (left > 0 ? left : 0) : (long)V * S);   // elements of this group that exist
    const T *w = static_cast<const T *>(J.w) + (long)co0 * S;
    const int n16 = n_el / V;
    for (int i = tid; i < n16; i += NT) slab4[i] = reinterpret_cast<const uint4 *>(w)[i];
    for (int i = n16 * V + tid; i < n_el; i += NT) slab[i] = w[i];
    __syncthreads();
    // filter element (output channel co0 + c, input channel ci, window position p); zero outside the tensor
    auto at = [&](int c, int ci, int p) -> T {
        const int i = c * S + ci * kk + p;
        return (ci < J.cin && i < n_el) ? slab[i] : (T)0.f;
    };
    union { uint4 u; T e[V]; } o;
    if (J.rw) {  // wf[co][ky][j], j = kx*rw + ci over a padded window row of KW elements
        const int jv = J.KW / V, n = V * k * jv;
        for (int i = tid; i < n; i += NT) {
            const int jg = i % jv, t = i / jv, ky = t % k, c = t / k;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const int j = jg * V + e, kx = j / J.rw, ci = j - kx * J.rw;
                o.e[e] = kx < k ? at(c, ci, ky * k + kx) : (T)0.f;
            }
            *reinterpret_cast<uint4 *>(static_cast<T *>(J.wf) + ((long)(co0 + c) * k + ky) * J.KW + jg * V) = o.u;
        }
        return;
    }
    if (J.wf) {  // wf[co][ky][kx][ci], with zeros up to the end of the last chunk
        const int cv = J.cinw / V, n = V * kk * cv;
        for (int i = tid; i < n; i += NT) {
            const int cg = i % cv, t = i / cv, pp = t % kk, c = t / kk;
#pragma unroll
            for (int e = 0; e < V; ++e) o.e[e] = at(c, cg * V + e, pp);
            const long at_f = J.fks ? direct_index(co0 + c, pp, cg * V, J.fks, J.fch, kk) : ((long)(co0 + c) * kk + pp) * J.cinp + cg * V;
            *reinterpret_cast<uint4 *>(static_cast<T *>(J.wf) + at_f) = o.u;
        }
    }
    if (J.wd) {  // wd[ci][ky'][kx'][co] = w[co][ci][k-1-ky'][k-1-kx']: this group's 16 bytes of every (ci, ky', kx')
        const int n = J.cinp * kk;
        for (int i = tid; i < n; i += NT) {
            const int pp = i % kk, ci = i / kk;
#pragma unroll
            for (int e = 0; e < V; ++e) o.e[e] = at(e, ci, kk - 1 - pp);
            const long at_d = J.dks ? direct_index(ci, pp, co0, J.dks, J.dch, kk) : ((long)ci * kk + pp) * J.coutp + co0;
            *reinterpret_cast<uint4 *>(static_cast<T *>(J.wd) + at_d) = o.u;
        }
    }
}

// The head of a forward pass in one launch: the first jobs.total workgroups pack filters, the others stage the images, 1024
// elements of work each.  The packing is a chain of few loads (13 us by itself for 172 workgroups), the staging a stream
// (20 us for 128 images of 3 x 224 x 224 in bf16); on two streams the events around them cost another 22 us.  Together, with
// four pixels per thread where the width allows: 54 -> 21 us.
template <typename T, int FORM, int PX> __global__ __launch_bounds__(1024) void head_kernel(PackJobs jobs, StageJob st)
{
    __shared__ uint4 slab4[4096];
    if (blockIdx.x < jobs.total) { pack_lds_block<T>(jobs, slab4); return; }
    const unsigned i = (blockIdx.x - jobs.total) * 1024u + threadIdx.x;
    if (i < st.total) stage_one<T, FORM, PX>(st, i);
}
template <typename T> static int launch_head_t(const PackJobs &jobs, StageJob st, hipStream_t s)
{
    // elements of work: 32-bit indices (the plan keeps an image tensor below 2^31 elements)
    const unsigned es = sizeof(T);
    int form = 0, px = 1;
    size_t work = st.src ? (size_t)st.B * st.H * st.W : 0;
    if (st.pc) {
        form = st.pc;
        const bool dwords2 = ((size_t)st.pad * st.pc * es) % 4 == 0 && ((size_t)st.Wp * st.pc * es) % 4 == 0 && ((size_t)2 * st.pc * es) % 4 == 0 && ((uintptr_t)st.dst & 3) == 0;
        if (dwords2 && st.W % 4 == 0 && ((uintptr_t)st.src & (4 * es - 1)) == 0) px = 4;
        else if (dwords2 && st.W % 2 == 0) px = 2;
        work /= (size_t)px;
    } else if (st.src) {
        work *= (size_t)(st.Cp / (int)(16 / es));
    }
    if (work > 0x7fffffffu) return -1;
    st.total = (unsigned)work;
    if (st.src) {
        st.dHW = make_fastdiv((uint32_t)(st.H * st.W)); st.dH = make_fastdiv((uint32_t)st.H); st.dWq = make_fastdiv((uint32_t)(st.W / px));
    }
    const unsigned blocks = jobs.total + (st.total + 1023u) / 1024u;
    if (blocks == 0) return 0;
#define ASGD_HEAD(F, P) if (form == F && px == P) { hipLaunchKernelGGL((head_kernel<T, F, P>), dim3(blocks), dim3(1024), 0, s, jobs, st); return launch_ok(); }
    ASGD_HEAD(0, 1)
    ASGD_HEAD(1, 1) ASGD_HEAD(1, 2) ASGD_HEAD(1, 4)
    ASGD_HEAD(2, 1) ASGD_HEAD(2, 2) ASGD_HEAD(2, 4)
    ASGD_HEAD(3, 1) ASGD_HEAD(3, 2) ASGD_HEAD(3, 4)
    ASGD_HEAD(4, 1) ASGD_HEAD(4, 2) ASGD_HEAD(4, 4)
#undef ASGD_HEAD
    return -1;
}

int launch_head(int dtype, PackJobs &jobs, const StageJob &st, hipStream_t s)
{
    if (st.src && ((st.pc && (st.C > st.pc || st.pc > 4)) || (size_t)st.B * st.H * st.W > 0x7fffffffu)) return -1;
    const auto head = [&](const PackJobs &pack) { return dtype == kBF16 ? launch_head_t<bf16_t>(pack, st, s) : launch_head_t<float>(pack, st, s); };
    PackJobs none;
    none.n = 0; none.total = 0;
    if (jobs.n == 0) return head(none);
    for (int q = 0; q < jobs.n; ++q) { PackJob &J = jobs.j[q]; J.cinw = J.fks ? J.fch * J.fks * 16 : J.cinp; }
    // the LDS form, if every layer qualifies
    {
        const size_t es = dtype_size(dtype), V = 16 / es;
        bool ok = jobs.n > 0;
        size_t blocks = 0;
        for (int q = 0; q < jobs.n && ok; ++q) {
            const PackJob &J = jobs.j[q];
            const size_t S = (size_t)J.cin * J.k * J.k;
            ok = V * S * es <= 65536 && (((uintptr_t)J.w | (uintptr_t)J.wf | (uintptr_t)J.wd) & 15) == 0 && J.coutp % 8 == 0 && J.cinp % 8 == 0 &&
                 (J.wf || J.wd) && (!J.rw || (J.wf && J.KW % 8 == 0 && J.rw > 0));
            blocks += (size_t)J.coutp / V;
        }
        if (ok && blocks <= 0x7fffffffull) {
            unsigned start = 0;
            for (int q = 0; q < jobs.n; ++q) { jobs.j[q].start = start; start += (unsigned)(jobs.j[q].coutp / (int)V); }
            jobs.total = start;
            return head(jobs);
        }
    }
    if (head(none) != 0) return -1;
    size_t total = 0;
    for (int q = 0; q < jobs.n; ++q) {
        PackJob &J = jobs.j[q];
        const size_t full = J.rw ? (size_t)J.coutp * J.k * J.KW : (size_t)J.coutp * J.k * J.k * J.cinp;
        const size_t nf = !J.wf ? 0 : J.rw ? full : full / J.cinp * J.cinw;
        const size_t nd = (!J.rw && J.wd) ? full : 0;
        if (nf + nd > 0xffffffffull || (nf & 7)) return -1;   // cinp, cinw, coutp and KW are multiples of 8
        J.start = (unsigned)total; J.nf = (unsigned)nf;
        total += (nf + nd) / 8;                                 // in groups of 8 elements
    }
    if (total == 0) return 0;
    jobs.total = (unsigned)total;
    const unsigned blocks = blocks_for(total, 256);
    if (dtype == kBF16) hipLaunchKernelGGL(pack_conv_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, jobs);
    else hipLaunchKernelGGL(pack_conv_kernel<float>, dim3(blocks), dim3(256), 0, s, jobs);
    return launch_ok();
}

// ---------------------------------------------------------------- max pooling
// Workgroup ids go round-robin over the 8 XCDs; neighbouring pixels share pooling windows, so each XCD is given a
// contiguous range of blocks (and its L2 fetches a window row once instead of every XCD fetching it).
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t nb)
{
    const uint32_t q = nb >> 3, r = nb & 7, x = b & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}
__device__ __forceinline__ uint32_t xcd_block() { return xcd_block(blockIdx.x, gridDim.x); }
// thread index -> (channel group, x, y, image) by three multiply-shift divisions (the index fits 31 bits)
struct PoolIndex { FastDiv dcv, dw, dh; int cv, w, h; };
static PoolIndex make_pool_index(int cv, int w, int h)
{
    return PoolIndex{make_fastdiv((uint32_t)cv), make_fastdiv((uint32_t)w), make_fastdiv((uint32_t)h), cv, w, h};
}
__device__ __forceinline__ void pool_decode(uint32_t i, const PoolIndex &p, int &cg, int &x, int &y, int &n)
{
    uint32_t t = fdiv32(i, p.dcv); cg = (int)(i - t * p.cv);
    uint32_t u = fdiv32(t, p.dw); x = (int)(t - u * p.w);
    n = (int)fdiv32(u, p.dh); y = (int)(u - (uint32_t)n * p.h);
}
// One thread owns VEC consecutive channels (16 bytes) of one output pixel.
template <typename T> struct Vec16 {
    static constexpr int N = 16 / sizeof(T);
    union { uint4 u; T e[16 / sizeof(T)]; };
};

// The first maximum of P values per channel in their order (a NaN counts only where it is the first value), and its index, one byte
// per channel.  KEYS: 16-bit data that is not negative, as after a ReLU, sorts as unsigned integers; value and 15 - index in one
// word make one v_max3 out of six compares and selects (96 channels 55 x 55, 128 images, windows of 3: 22.8 -> 16.2 us, 256 channels
// 27 x 27 14.6 -> 10.5).  Keys above infinity's (a NaN, a negative value after all, -0) take the compares.
template <typename T, int P, bool KEYS> __device__ __forceinline__ void first_max(const Vec16<T> (&v)[P], Vec16<T> &o, uint64_t &pos)
{
    constexpr int V = Vec16<T>::N;
    if constexpr (KEYS) {
        static_assert(sizeof(T) == 2 && P <= 15, "a key is 16 bits of value over 15 - index");
        uint32_t m[V], worst = 0;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            uint32_t k[P];
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const uint32_t w = e / 2 == 0 ? v[j].u.x : e / 2 == 1 ? v[j].u.y : e / 2 == 2 ? v[j].u.z : v[j].u.w;
                k[j] = (e & 1 ? w & 0xFFFF0000u : w << 16) | (uint32_t)(15 - j);
            }
            m[e] = k[0];
#pragma unroll
            for (int j = 1; j + 1 < P; j += 2) m[e] = max(max(m[e], k[j]), k[j + 1]);
            if (P % 2 == 0) m[e] = max(m[e], k[P - 1]);
            worst = max(worst, m[e]);
        }
        if (worst <= 0x7F80FFFFu) {
            // v_perm_b32: selector bytes 0-3 take the second operand's, 4-7 the first one's
            o.u = make_uint4(__builtin_amdgcn_perm(m[1], m[0], 0x07060302u), __builtin_amdgcn_perm(m[3], m[2], 0x07060302u),
                             __builtin_amdgcn_perm(m[5], m[4], 0x07060302u), __builtin_amdgcn_perm(m[7], m[6], 0x07060302u));
            const uint32_t lo = __builtin_amdgcn_perm(__builtin_amdgcn_perm(m[3], m[2], 0x0C0C0400u), __builtin_amdgcn_perm(m[1], m[0], 0x0C0C0400u), 0x05040100u);
            const uint32_t hi = __builtin_amdgcn_perm(__builtin_amdgcn_perm(m[7], m[6], 0x0C0C0400u), __builtin_amdgcn_perm(m[5], m[4], 0x0C0C0400u), 0x05040100u);
            pos = (lo ^ 0x0F0F0F0Fu) | (uint64_t)(hi ^ 0x0F0F0F0Fu) << 32;
            return;
        }
    }
    float best[V];
    uint32_t a[V];
#pragma unroll
    for (int j = 0; j < P; ++j) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float f = ldf(&v[j].e[e]);
            if (j == 0 || f > best[e]) { best[e] = f; a[e] = (uint32_t)j; }
        }
    }
    pos = 0;
#pragma unroll
    for (int e = 0; e < V; ++e) { stf(&o.e[e], best[e]); pos |= (uint64_t)a[e] << (8 * e); }
}

// KC > 0: window size known at compile time, so the k*k loads of a thread are all issued before the first compare.
template <typename T, int KC, bool KEYS>
__global__ __launch_bounds__(256) void pool_fwd_kernel(const T *__restrict__ x, T *__restrict__ y, uint8_t *__restrict__ arg, int B, int H, int W,
                                                     int Cp, int k_rt, int stride, int Ho, int Wo, PoolIndex pi)
{
    constexpr int V = Vec16<T>::N;
    const int k = KC > 0 ? KC : k_rt;
    const uint32_t i = xcd_block() * 256u + threadIdx.x;
    if (i >= (uint32_t)B * Ho * Wo * pi.cv) return;
    int cg, px, py, n;
    pool_decode(i, pi, cg, px, py, n);
    const int c0 = cg * V;
    const T *win = x + (((long)n * H + py * stride) * W + px * stride) * Cp + c0;
    Vec16<T> o;
    uint64_t packed = 0;
    if constexpr (KC > 0) {
        Vec16<T> v[KC * KC];
#pragma unroll
        for (int p = 0; p < KC * KC; ++p) v[p].u = *reinterpret_cast<const uint4 *>(win + ((long)(p / KC) * W + (p % KC)) * Cp);
        first_max<T, KC * KC, KEYS>(v, o, packed);
    } else {
        float best[V];
        uint8_t a[V];
        for (int ky = 0; ky < k; ++ky)
            for (int kx = 0; kx < k; ++kx) {
                Vec16<T> v;
                v.u = *reinterpret_cast<const uint4 *>(win + ((long)ky * W + kx) * Cp);
                const int pos = ky * k + kx;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float f = ldf(&v.e[e]);
                    if (pos == 0 || f > best[e]) { best[e] = f; a[e] = (uint8_t)pos; }
                }
            }
#pragma unroll
        for (int e = 0; e < V; ++e) { stf(&o.e[e], best[e]); packed |= (uint64_t)a[e] << (8 * e); }
    }
    const long off = (((long)n * Ho + py) * Wo + px) * Cp + c0;
    *reinterpret_cast<uint4 *>(y + off) = o.u;
    if (V == 8) *reinterpret_cast<uint64_t *>(arg + off) = packed;
    else *reinterpret_cast<uint32_t *>(arg + off) = (uint32_t)packed;
}

template <typename T, bool KEYS>
static void launch_pool_fwd_t(const void *x, void *y, uint8_t *arg, int B, int H, int W, int Cp, int k, int stride, int Ho, int Wo, unsigned blocks,
                              hipStream_t s)
{
    const T *xx = static_cast<const T *>(x); T *yy = static_cast<T *>(y);
    const PoolIndex pi = make_pool_index(Cp / (16 / (int)sizeof(T)), Wo, Ho);
    if (k == 3) hipLaunchKernelGGL((pool_fwd_kernel<T, 3, KEYS>), dim3(blocks), dim3(256), 0, s, xx, yy, arg, B, H, W, Cp, k, stride, Ho, Wo, pi);
    else if (k == 2) hipLaunchKernelGGL((pool_fwd_kernel<T, 2, KEYS>), dim3(blocks), dim3(256), 0, s, xx, yy, arg, B, H, W, Cp, k, stride, Ho, Wo, pi);
    else hipLaunchKernelGGL((pool_fwd_kernel<T, 0, false>), dim3(blocks), dim3(256), 0, s, xx, yy, arg, B, H, W, Cp, k, stride, Ho, Wo, pi);
}
int launch_pool_fwd(int dtype, const void *x, int nonneg, void *y, uint8_t *arg, int B, int H, int W, int Cp, int k, int stride, hipStream_t s)
{
    const int Ho = (H - k) / stride + 1, Wo = (W - k) / stride + 1;
    const int V = dtype == kBF16 ? 8 : 4;
    if ((size_t)B * Ho * Wo * (Cp / V) > 0x7fffffffu) return -1;
    const unsigned blocks = blocks_for((size_t)B * Ho * Wo * (Cp / V), 256);
    if (dtype == kBF16 && nonneg) launch_pool_fwd_t<bf16_t, true>(x, y, arg, B, H, W, Cp, k, stride, Ho, Wo, blocks, s);
    else if (dtype == kBF16) launch_pool_fwd_t<bf16_t, false>(x, y, arg, B, H, W, Cp, k, stride, Ho, Wo, blocks, s);
    else launch_pool_fwd_t<float, false>(x, y, arg, B, H, W, Cp, k, stride, Ho, Wo, blocks, s);
    return launch_ok();
}

// Gather form: an input pixel sums, in (py, px) order, the gradients of the
// windows whose recorded maximum it is; then, if asked, the ReLU mask of the layer below.
// TWO: at most two windows per axis cover a pixel (k <= 2*stride); the four candidate windows are then
// fetched up front, with the out-of-range ones masked, instead of in a loop whose loads wait for each other.
template <typename T, bool TWO>
__global__ __launch_bounds__(256) void pool_bwd_kernel(const T *__restrict__ dy, const uint8_t *__restrict__ arg, const T *__restrict__ x, int relu,
                                                     T *__restrict__ dx, int B, int H, int W, int Cp, int k, int stride, int Ho, int Wo,
                                                     PoolIndex pi, FastDiv dstride)
{
    constexpr int V = Vec16<T>::N;
    const uint32_t i = xcd_block() * 256u + threadIdx.x;
    if (i >= (uint32_t)B * H * W * pi.cv) return;
    int cg, ix, iy, n;
    pool_decode(i, pi, cg, ix, iy, n);
    const int c0 = cg * V;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    int py0 = iy - k + 1; py0 = py0 <= 0 ? 0 : (int)fdiv32((uint32_t)(py0 + stride - 1), dstride);
    int px0 = ix - k + 1; px0 = px0 <= 0 ? 0 : (int)fdiv32((uint32_t)(px0 + stride - 1), dstride);
    const int py1 = min((int)fdiv32((uint32_t)iy, dstride), Ho - 1), px1 = min((int)fdiv32((uint32_t)ix, dstride), Wo - 1);
    auto add = [&](const Vec16<T> &g, uint64_t a8, int pos, bool ok) {
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (ok && (int)((a8 >> (8 * e)) & 0xff) == pos) acc[e] += ldf(&g.e[e]);
    };
    if constexpr (TWO) {
        Vec16<T> g[4];
        uint64_t a8[4];
        int pos[4];
        bool ok[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // (py0, px0), (py0, px0+1), (py0+1, px0), (py0+1, px0+1)
            const int py = py0 + (q >> 1), px = px0 + (q & 1);
            ok[q] = py <= py1 && px <= px1;
            pos[q] = (iy - py * stride) * k + (ix - px * stride);
            const long off = (((long)n * Ho + py) * Wo + px) * Cp + c0;
            // windows that do not cover the pixel (more than half of the candidates for 3/2 pooling) are not fetched:
            // the kernel is bound by what it pulls out of L2, not by HBM
            g[q].u = make_uint4(0u, 0u, 0u, 0u);
            a8[q] = 0;
            if (ok[q]) {
                g[q].u = *reinterpret_cast<const uint4 *>(dy + off);
                if (V == 8) a8[q] = *reinterpret_cast<const uint64_t *>(arg + off);
                else a8[q] = *reinterpret_cast<const uint32_t *>(arg + off);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) add(g[q], a8[q], pos[q], ok[q]);
    } else {
        for (int py = py0; py <= py1; ++py)
            for (int px = px0; px <= px1; ++px) {
                const long off = (((long)n * Ho + py) * Wo + px) * Cp + c0;
                Vec16<T> g;
                g.u = *reinterpret_cast<const uint4 *>(dy + off);
                uint64_t a8;   // the V recorded positions of this window, one byte each
                if (V == 8) a8 = *reinterpret_cast<const uint64_t *>(arg + off);
                else a8 = *reinterpret_cast<const uint32_t *>(arg + off);
                add(g, a8, (iy - py * stride) * k + (ix - px * stride), true);
            }
    }
    const long off = (((long)n * H + iy) * W + ix) * Cp + c0;
    Vec16<T> o;
    if (relu) {
        Vec16<T> xv;
        xv.u = *reinterpret_cast<const uint4 *>(x + off);
#pragma unroll
        for (int e = 0; e < V; ++e) stf(&o.e[e], ldf(&xv.e[e]) > 0.f ? acc[e] : 0.f);
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) stf(&o.e[e], acc[e]);
    }
    *reinterpret_cast<uint4 *>(dx + off) = o.u;
}

// What the 2 x 2 blocks of input pixels of a pool with stride 2 and windows of 2 or 3 need of the pool's side: gradients and
// positions of the four windows (jy-1, jx-1), (jy-1, jx), (jy, jx-1), (jy, jx), by range-checked loads without a branch: a window
// outside the grid reads as a gradient of zero (at position 0).  at: element offset of window (jy-1, jx-1) from the start of
// the ranges, which hold less than 2 GiB.
template <typename T> struct PoolWindows {
    Vec16<T> g[4];
    uint2 a8[4];
    static __device__ __forceinline__ bool inside(int q, int jy, int jx, int Ho, int Wo)
    {
        const bool up = jy > 0 && jy <= Ho, down = (unsigned)jy < (unsigned)Ho, left = jx > 0 && jx <= Wo, right = (unsigned)jx < (unsigned)Wo;
        return (q < 2 ? up : down) && (q & 1 ? right : left);
    }
    __device__ __forceinline__ void load_positions(__amdgpu_buffer_rsrc_t arg, unsigned at, int jy, int jx, int Ho, int Wo, int Cp)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned o = inside(q, jy, jx, Ho, Wo) ? at + (unsigned)((q >> 1) * Wo * Cp + (q & 1) * Cp) : kInv;
            if constexpr (sizeof(T) == 2) {
                typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(arg, (int)o, 0, 0);
                a8[q] = make_uint2(v.x, v.y);
            } else {
                a8[q] = make_uint2(__builtin_amdgcn_raw_buffer_load_b32(arg, (int)o, 0, 0), 0u);
            }
        }
    }
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t dy, __amdgpu_buffer_rsrc_t arg, unsigned at, int jy, int jx, int Ho, int Wo, int Cp)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            g[q].u = buf_ld16(dy, inside(q, jy, jx, Ho, Wo) ? (at + (unsigned)((q >> 1) * Wo * Cp + (q & 1) * Cp)) * (unsigned)sizeof(T) : kInv);
        load_positions(arg, at, jy, jx, Ho, Wo, Cp);
    }
    // the gradients of the block's pixels (0, 0), (0, 1), (1, 0), (1, 1), added in window order
    template <int K> __device__ __forceinline__ void sums(float (&acc)[4][Vec16<T>::N]) const
    {
        constexpr int V = Vec16<T>::N;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float ge[4];
            unsigned pos[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ge[q] = ldf(&g[q].e[e]);
                pos[q] = ((e < 4 ? a8[q].x : a8[q].y) >> (8 * (e & 3))) & 0xffu;
            }
#pragma unroll
            for (int b = 0; b < 4; ++b) {   // pixel (by, bx) sits at (by + 2*(1 - wy), bx + 2*(1 - wx)) in window q = (wy, wx)
                float t = 0.f;
                bool any = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int ry = (b >> 1) + 2 * (1 - (q >> 1)), rx = (b & 1) + 2 * (1 - (q & 1));
                    if (ry < K && rx < K) {
                        const float v = pos[q] == (unsigned)(ry * K + rx) ? ge[q] : 0.f;
                        t = any ? t + v : v;
                        any = true;
                    }
                }
                acc[b][e] = t;
            }
        }
    }
};
__device__ __forceinline__ __amdgpu_buffer_rsrc_t byte_range(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(unsigned)(bytes < 0x7fffffffu ? bytes : 0x7fffffffu), 0x00020000);
}

// Stride 2, windows of 2 or 3: a thread owns a 2 x 2 block of input pixels (rows 2*jy, 2*jy+1, columns 2*jx,
// 2*jx+1).  Exactly the four windows (jy-1 .. jy) x (jx-1 .. jx) can cover it: window (jy, jx) covers all four
// pixels, the two neighbours above / to the left cover the pixels of the block's first row / column (3 x 3
// only), the diagonal one its first pixel.  The four windows are fetched once for the four pixels (the
// pixel-per-thread form fetches 2.25 windows per pixel) and each recorded position is decoded once.  The sums
// run over the windows in the same order as in the general kernel, so the results are the same bit for bit.
// If bands is given, the block also leaves the column sums of what it stored (the gradient at the output of the
// convolution below, whose bias gradient they are part of) in bands[column][block]: the values as stored (rounded
// to the element type), added per thread over its pixels, then over the block's threads in thread order.
template <typename T, int K>
__device__ __forceinline__ void pool_bwd_s2_block(const T *__restrict__ dy, const uint8_t *__restrict__ arg, const T *__restrict__ x, int relu,
                                                  T *__restrict__ dx, int B, int H, int W, int Cp, int Ho, int Wo, const PoolIndex &pi,
                                                  float *__restrict__ bands, uint32_t blk, uint32_t blocks, float *part)
{
    constexpr int V = Vec16<T>::N;
    const uint32_t i = blk * 256u + threadIdx.x;
    const bool live = i < (uint32_t)B * pi.h * pi.w * pi.cv;
    if (!live && bands == nullptr) return;
    int cg, jx, jy, n;
    pool_decode(live ? i : 0u, pi, cg, jx, jy, n);
    if (!live) { jy = -4; jx = -4; }   // no window, no pixel: contributes zeros to the band sums
    const int c0 = cg * V;
    // ranges that start with the image of the block's first thread
    const int n0 = (int)fdiv32(fdiv32(fdiv32(blk * 256u, pi.dcv), pi.dw), pi.dh);
    const size_t before = (size_t)n0 * Ho * Wo * Cp, behind = (size_t)(B - n0) * Ho * Wo * Cp;
    PoolWindows<T> win;
    win.load(byte_range(dy + before, behind * sizeof(T)), byte_range(arg + before, behind),
             (unsigned)((((n - n0) * Ho + jy - 1) * Wo + jx - 1) * Cp + c0), jy, jx, Ho, Wo, Cp);
    float acc[4][V];
    win.template sums<K>(acc);
    float colsum[V];
#pragma unroll
    for (int e = 0; e < V; ++e) colsum[e] = 0.f;
    const long at = (((long)n * H + 2 * jy) * W + 2 * jx) * Cp + c0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if ((unsigned)(2 * jy + (b >> 1)) < (unsigned)H && (unsigned)(2 * jx + (b & 1)) < (unsigned)W) {
            const long off = at + (long)((b >> 1) * W + (b & 1)) * Cp;
            Vec16<T> o;
            if (relu) {
                Vec16<T> xv;
                xv.u = *reinterpret_cast<const uint4 *>(x + off);
#pragma unroll
                for (int e = 0; e < V; ++e) stf(&o.e[e], ldf(&xv.e[e]) > 0.f ? acc[b][e] : 0.f);
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) stf(&o.e[e], acc[b][e]);
            }
            *reinterpret_cast<uint4 *>(dx + off) = o.u;
#pragma unroll
            for (int e = 0; e < V; ++e) colsum[e] += ldf(&o.e[e]);
        }
    }
    if (bands == nullptr) return;
    // thread t of the block holds channel group (blk * 256 + t) % cv: column c adds the threads of its group in order
#pragma unroll
    for (int e = 0; e < V; ++e) part[threadIdx.x * V + e] = colsum[e];
    __syncthreads();
    const int cv = pi.cv;
    const int g0 = (int)((blk * 256u) % (uint32_t)cv);   // group of thread 0
    for (int c = threadIdx.x; c < Cp; c += 256) {
        const int gc = c / V, e = c - gc * V;
        float t = 0.f;
        for (int j = (gc - g0 + cv) % cv; j < 256; j += cv) t += part[j * V + e];
        bands[(long)c * blocks + blk] = t;
    }
}
template <typename T, int K>
__global__ __launch_bounds__(256) void pool_bwd_s2_kernel(const T *__restrict__ dy, const uint8_t *__restrict__ arg, const T *__restrict__ x, int relu,
                                                        T *__restrict__ dx, int B, int H, int W, int Cp, int Ho, int Wo, PoolIndex pi,
                                                        float *__restrict__ bands)
{
    __shared__ float part[256 * Vec16<T>::N];
    pool_bwd_s2_block<T, K>(dy, arg, x, relu, dx, B, H, W, Cp, Ho, Wo, pi, bands, xcd_block(), gridDim.x, part);
}
// The same with a reduction of partial sums (its first red.blocks workgroups).
template <typename T, int K>
__global__ __launch_bounds__(256) void pool_bwd_s2_reduce_kernel(const T *__restrict__ dy, const uint8_t *__restrict__ arg, const T *__restrict__ x, int relu,
                                                               T *__restrict__ dx, int B, int H, int W, int Cp, int Ho, int Wo, PoolIndex pi,
                                                               float *__restrict__ bands, Reduction red)
{
    __shared__ union { float part[256 * Vec16<T>::N]; ReduceShared red; } sh;
    if (blockIdx.x < red.blocks) reduce_block<T>(red, blockIdx.x, sh.red);
    else pool_bwd_s2_block<T, K>(dy, arg, x, relu, dx, B, H, W, Cp, Ho, Wo, pi, bands, xcd_block(blockIdx.x - red.blocks, gridDim.x - red.blocks),
                                 gridDim.x - red.blocks, sh.part);
}

// Where pool_bwd_s2_kernel runs: a block's 256 threads see two images, or several small ones, in one range of 2 GiB.
static bool pool_bwd_blocks(int H, int W, int Cp, int es, int k, int stride)
{
    return stride == 2 && (k == 2 || k == 3) && (size_t)H * W * Cp * es < ((size_t)1 << 30);
}
template <typename T>
static void launch_pool_bwd_t(const void *dy, const uint8_t *arg, const void *x, int relu, void *dx, int B, int H, int W, int Cp, int k, int stride,
                              int Ho, int Wo, unsigned blocks, float *bands, const Reduction *beside, hipStream_t s)
{
    const T *d = static_cast<const T *>(dy), *xx = static_cast<const T *>(x); T *o = static_cast<T *>(dx);
    if (pool_bwd_blocks(H, W, Cp, (int)sizeof(T), k, stride)) {
        const int Hb = (H + 1) / 2, Wb = (W + 1) / 2, cv = Cp / (16 / (int)sizeof(T));
        const PoolIndex pb = make_pool_index(cv, Wb, Hb);
        const unsigned nb = blocks_for((size_t)B * Hb * Wb * cv, 256);
        if (beside) {
            const dim3 grid(nb + beside->blocks);
            if (k == 3) hipLaunchKernelGGL((pool_bwd_s2_reduce_kernel<T, 3>), grid, dim3(256), 0, s, d, arg, xx, relu, o, B, H, W, Cp, Ho, Wo, pb, bands, *beside);
            else hipLaunchKernelGGL((pool_bwd_s2_reduce_kernel<T, 2>), grid, dim3(256), 0, s, d, arg, xx, relu, o, B, H, W, Cp, Ho, Wo, pb, bands, *beside);
            return;
        }
        if (k == 3) hipLaunchKernelGGL((pool_bwd_s2_kernel<T, 3>), dim3(nb), dim3(256), 0, s, d, arg, xx, relu, o, B, H, W, Cp, Ho, Wo, pb, bands);
        else hipLaunchKernelGGL((pool_bwd_s2_kernel<T, 2>), dim3(nb), dim3(256), 0, s, d, arg, xx, relu, o, B, H, W, Cp, Ho, Wo, pb, bands);
        return;
    }
    const PoolIndex pi = make_pool_index(Cp / (16 / (int)sizeof(T)), W, H);
    const FastDiv ds = make_fastdiv((uint32_t)stride);
    if (k <= 2 * stride) hipLaunchKernelGGL((pool_bwd_kernel<T, true>), dim3(blocks), dim3(256), 0, s, d, arg, xx, relu, o, B, H, W, Cp, k, stride, Ho, Wo, pi, ds);
    else hipLaunchKernelGGL((pool_bwd_kernel<T, false>), dim3(blocks), dim3(256), 0, s, d, arg, xx, relu, o, B, H, W, Cp, k, stride, Ho, Wo, pi, ds);
}
// Number of column-sum bands the pooling backward pass can leave behind (0: this shape runs a kernel that cannot).
long pool_bwd_bands(int dtype, int B, int H, int W, int Cp, int k, int stride)
{
    if (!pool_bwd_blocks(H, W, Cp, (int)dtype_size(dtype), k, stride)) return 0;
    const int V = dtype == kBF16 ? 8 : 4;
    return (long)blocks_for((size_t)B * ((H + 1) / 2) * ((W + 1) / 2) * (Cp / V), 256);
}
int launch_pool_bwd(int dtype, const void *dy, const uint8_t *arg, const void *x, int relu, void *dx, int B, int H, int W, int Cp, int k, int stride,
                    float *bands, const Reduction *beside, hipStream_t s)
{
    const int Ho = (H - k) / stride + 1, Wo = (W - k) / stride + 1;
    const int V = dtype == kBF16 ? 8 : 4;
    if ((size_t)B * H * W * (Cp / V) > 0x7fffffffu) return -1;
    if ((bands || beside) && pool_bwd_bands(dtype, B, H, W, Cp, k, stride) == 0) return -1;
    const unsigned blocks = blocks_for((size_t)B * H * W * (Cp / V), 256);
    if (dtype == kBF16) launch_pool_bwd_t<bf16_t>(dy, arg, x, relu, dx, B, H, W, Cp, k, stride, Ho, Wo, blocks, bands, beside, s);
    else launch_pool_bwd_t<float>(dy, arg, x, relu, dx, B, H, W, Cp, k, stride, Ho, Wo, blocks, bands, beside, s);
    return launch_ok();
}

// ---------------------------------------------------------------- the pool under the first fully-connected layer
// Its output is wanted in the order (channel, row, column) of that layer's weights, and its gradient arrives in it: both kernels
// turn a chunk of channels of one image around in LDS, so that the flat side is one contiguous run and neither the
// channel-last tensor nor its gradient goes to memory.  Bound by the latency of their loads.  128 images, 13 x 13 pools of 3 over 256
// channels in bf16: pool and flatten 11.6 us, here 5.2; unflatten and pool 16.6, here 12.2.
struct PoolFlat {
    int H, W, C, Cp, Ho, Wo, hw, cv, groups, chunks, lanes, Hb, Wb;   // hw: pooled pixels; groups of 16 bytes of channels a block takes
    FastDiv dgroups, dchunks, dWo, dWb;
};
constexpr int kPoolFlatLds = 32 << 10;
template <typename T, int K, bool KEYS>
__global__ __launch_bounds__(256) void pool_flat_fwd_kernel(const T *__restrict__ x, T *__restrict__ flat, uint8_t *__restrict__ arg, PoolFlat p)
{
    constexpr int V = Vec16<T>::N;
    extern __shared__ uint4 lds[];
    T *tile = reinterpret_cast<T *>(lds);   // [channel][pooled pixel]
    const uint32_t blk = xcd_block();
    const int n = (int)fdiv32(blk, p.dchunks), g0 = ((int)blk - n * p.chunks) * p.groups;
    for (int i = threadIdx.x; i < p.hw * p.groups; i += 256) {
        const int pix = (int)fdiv32((uint32_t)i, p.dgroups), g = i - pix * p.groups, c0 = (g0 + g) * V;
        if (c0 >= p.Cp) continue;
        const int py = (int)fdiv32((uint32_t)pix, p.dWo), px = pix - py * p.Wo;
        const T *win = x + (((long)n * p.H + 2 * py) * p.W + 2 * px) * p.Cp + c0;
        Vec16<T> v[K * K], o;
#pragma unroll
        for (int j = 0; j < K * K; ++j) v[j].u = *reinterpret_cast<const uint4 *>(win + ((long)(j / K) * p.W + j % K) * p.Cp);
        uint64_t packed;
        first_max<T, K * K, KEYS>(v, o, packed);
        uint8_t *a = arg + ((long)n * p.hw + pix) * p.Cp + c0;
        if (V == 8) *reinterpret_cast<uint64_t *>(a) = packed;
        else *reinterpret_cast<uint32_t *>(a) = (uint32_t)packed;
#pragma unroll
        for (int e = 0; e < V; ++e) tile[(g * V + e) * p.hw + pix] = o.e[e];
    }
    __syncthreads();
    // whole vectors: eight channels, and the net's flattened size, are multiples of 16 bytes
    const int count = min(p.groups * V, p.C - g0 * V) * p.hw / V;
    uint4 *out = reinterpret_cast<uint4 *>(flat + ((long)n * p.C + g0 * V) * p.hw);
    for (int i = threadIdx.x; i < count; i += 256) out[i] = lds[i];
}
template <typename T, int K>
__global__ __launch_bounds__(256) void pool_flat_bwd_kernel(const T *__restrict__ dflat, const T *__restrict__ flat, int relu, const uint8_t *__restrict__ arg,
                                                          T *__restrict__ dx, PoolFlat p, float *__restrict__ bands, int B)
{
    constexpr int V = Vec16<T>::N;
    extern __shared__ uint4 lds[];
    T *tile = reinterpret_cast<T *>(lds);
    const uint32_t blk = xcd_block();
    const int n = (int)fdiv32(blk, p.dchunks), g0 = ((int)blk - n * p.chunks) * p.groups, channels = p.groups * V;
    const int count = min(channels, p.C - g0 * V) * p.hw / V;
    const long at = ((long)n * p.C + g0 * V) * p.hw;
    const uint4 *src = reinterpret_cast<const uint4 *>(dflat + at), *val = reinterpret_cast<const uint4 *>(flat + at);
    for (int i = threadIdx.x; i < channels * p.hw / V; i += 256) {
        Vec16<T> d;
        d.u = make_uint4(0u, 0u, 0u, 0u);   // padding channels
        if (i < count) {
            d.u = src[i];
            if (relu) {   // that of the convolution under the pool, on the pooled value
                Vec16<T> f;
                f.u = val[i];
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (!(ldf(&f.e[e]) > 0.f)) stf(&d.e[e], 0.f);
            }
        }
        lds[i] = d.u;
    }
    __syncthreads();
    const int j0 = (int)fdiv32(threadIdx.x, p.dgroups), g = (int)threadIdx.x - j0 * p.groups, c0 = (g0 + g) * V;
    const bool live = j0 < p.lanes && c0 < p.Cp;
    const __amdgpu_buffer_rsrc_t ra = byte_range(arg + (size_t)n * p.hw * p.Cp, (size_t)p.hw * p.Cp);
    float colsum[V];
#pragma unroll
    for (int e = 0; e < V; ++e) colsum[e] = 0.f;
    for (int j = j0; live && j < p.Hb * p.Wb; j += p.lanes) {
        const int jy = (int)fdiv32((uint32_t)j, p.dWb), jx = j - jy * p.Wb;
        PoolWindows<T> win;
        win.load_positions(ra, (unsigned)(((jy - 1) * p.Wo + jx - 1) * p.Cp + c0), jy, jx, p.Ho, p.Wo, p.Cp);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int py = jy - 1 + (q >> 1), px = jx - 1 + (q & 1);
            const bool ok = (unsigned)py < (unsigned)p.Ho && (unsigned)px < (unsigned)p.Wo;
            const T *t = tile + g * V * p.hw + (ok ? py * p.Wo + px : 0);
#pragma unroll
            for (int e = 0; e < V; ++e) win.g[q].e[e] = ok ? t[e * p.hw] : (T)0.f;
        }
        float acc[4][V];
        win.template sums<K>(acc);
        const long off = (((long)n * p.H + 2 * jy) * p.W + 2 * jx) * p.Cp + c0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (2 * jy + (b >> 1) >= p.H || 2 * jx + (b & 1) >= p.W) continue;
            Vec16<T> o;
#pragma unroll
            for (int e = 0; e < V; ++e) { stf(&o.e[e], acc[b][e]); colsum[e] += ldf(&o.e[e]); }
            *reinterpret_cast<uint4 *>(dx + off + (long)((b >> 1) * p.W + (b & 1)) * p.Cp) = o.u;
        }
    }
    __syncthreads();
    float *part = reinterpret_cast<float *>(lds);   // [lane][channel]
    if (j0 < p.lanes) {
#pragma unroll
        for (int e = 0; e < V; ++e) part[j0 * channels + g * V + e] = colsum[e];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < channels && g0 * V + c < p.Cp; c += 256) {
        float t = 0.f;
        for (int j = 0; j < p.lanes; ++j) t += part[j * channels + c];
        bands[(long)(g0 * V + c) * B + n] = t;
    }
}
static bool pool_flat_plan(int dtype, int B, int H, int W, int C, int Cp, int k, int stride, PoolFlat &p, size_t &lds_fwd, size_t &lds_bwd)
{
    const int V = dtype == kBF16 ? 8 : 4;
    if (!pool_bwd_blocks(H, W, Cp, (int)dtype_size(dtype), k, stride) || H < k || W < k) return false;
    p.H = H; p.W = W; p.C = C; p.Cp = Cp; p.Ho = (H - k) / 2 + 1; p.Wo = (W - k) / 2 + 1; p.hw = p.Ho * p.Wo; p.cv = Cp / V;
    if ((long)C * p.hw % 8 != 0 || (long)p.hw * 16 > kPoolFlatLds) return false;
    p.groups = std::max(1, std::min(p.cv, 256 / p.hw));   // one pooled pixel and group a thread
    p.chunks = (p.cv + p.groups - 1) / p.groups;
    p.lanes = 256 / p.groups; p.Hb = (H + 1) / 2; p.Wb = (W + 1) / 2;
    if ((long)B * p.chunks > 0x7fffffffL) return false;
    lds_fwd = (size_t)p.groups * p.hw * 16;
    lds_bwd = std::max(lds_fwd, (size_t)p.lanes * p.groups * V * 4);
    p.dgroups = make_fastdiv(p.groups); p.dchunks = make_fastdiv(p.chunks); p.dWo = make_fastdiv(p.Wo); p.dWb = make_fastdiv(p.Wb);
    return true;
}
long pool_flat_bands(int dtype, int B, int H, int W, int C, int Cp, int k, int stride, bool forked, bool always)
{
    PoolFlat p;
    size_t f, b;
    if (!pool_flat_plan(dtype, B, H, W, C, Cp, k, stride, p, f, b)) return 0;
    const long blocks = (long)B * p.chunks, reads = (long)p.hw * k * k, V = dtype == kBF16 ? 8 : 4;
    // A block that makes many pooled pixels in turn, one 16-byte group of each, is long: the two launches that the separate kernels
    // cost (about 8 us) pay for 2200 reads of a group, for 3400 where a pixel is two or three groups and for 4500 where it is one;
    // beyond, half the CUs have to have a block, and more of them the more a block reads (four-byte data and windows of 3 over large
    // grids gain nothing).  Beside a weight gradient on the side stream a long block costs less and a launch more: up to 6500 reads, or
    // four groups a pixel, one kernel.  A pass with separate kernels / here, us, bf16, 64 channels: pools of 2, 20 x 20 1 image
    // 53 / 55, 64 images 90 / 79, 45 x 45 78 / 99 and 221 / 182; pools of 3, 32 x 32 63 / 85 and 142 / 136; with the side stream 27 x 25
    // pools of 2 4 images 137 / 125, 28 x 20 pools of 3 2 images 149 / 139, 44 x 40 146 / 163.  Over 320 passes without and 150 with the side
    // stream the choice is at most 1.05 of the better one.
    const long few = p.cv == 1 ? 4500 : p.cv <= 3 ? 3400 : 2200;
    const bool apart = forked ? reads > 6500 && p.cv > 4 && blocks < std::max(128L, reads / 72)
                              : reads > few && (blocks < std::max(128L, reads / 36) || (V == 4 && k == 3 && reads > 4600));
    return apart && !always ? 0 : B;
}
template <typename T, bool KEYS> static void launch_pool_flat_fwd_t(const void *x, void *flat, uint8_t *arg, int B, int k, const PoolFlat &p, size_t lds, hipStream_t s)
{
    const dim3 grid((unsigned)(B * p.chunks));
    if (k == 3) hipLaunchKernelGGL((pool_flat_fwd_kernel<T, 3, KEYS>), grid, dim3(256), lds, s, static_cast<const T *>(x), static_cast<T *>(flat), arg, p);
    else hipLaunchKernelGGL((pool_flat_fwd_kernel<T, 2, KEYS>), grid, dim3(256), lds, s, static_cast<const T *>(x), static_cast<T *>(flat), arg, p);
}
int launch_pool_flat_fwd(int dtype, const void *x, int nonneg, void *flat, uint8_t *arg, int B, int H, int W, int C, int Cp, int k, hipStream_t s)
{
    PoolFlat p;
    size_t lf, lb;
    if (!pool_flat_plan(dtype, B, H, W, C, Cp, k, 2, p, lf, lb)) return -1;
    if (dtype == kBF16 && nonneg) launch_pool_flat_fwd_t<bf16_t, true>(x, flat, arg, B, k, p, lf, s);
    else if (dtype == kBF16) launch_pool_flat_fwd_t<bf16_t, false>(x, flat, arg, B, k, p, lf, s);
    else launch_pool_flat_fwd_t<float, false>(x, flat, arg, B, k, p, lf, s);
    return launch_ok();
}
template <typename T>
static void launch_pool_flat_bwd_t(const void *dflat, const void *flat, int relu, const uint8_t *arg, void *dx, int B, int k, const PoolFlat &p, float *bands,
                                   size_t lds, hipStream_t s)
{
    const dim3 grid((unsigned)(B * p.chunks));
    const T *d = static_cast<const T *>(dflat), *f = static_cast<const T *>(flat);
    if (k == 3) hipLaunchKernelGGL((pool_flat_bwd_kernel<T, 3>), grid, dim3(256), lds, s, d, f, relu, arg, static_cast<T *>(dx), p, bands, B);
    else hipLaunchKernelGGL((pool_flat_bwd_kernel<T, 2>), grid, dim3(256), lds, s, d, f, relu, arg, static_cast<T *>(dx), p, bands, B);
}
int launch_pool_flat_bwd(int dtype, const void *dflat, const void *flat, int relu, const uint8_t *arg, void *dx, int B, int H, int W, int C, int Cp, int k,
                         float *bands, hipStream_t s)
{
    PoolFlat p;
    size_t lf, lb;
    if (!pool_flat_plan(dtype, B, H, W, C, Cp, k, 2, p, lf, lb)) return -1;
    if (dtype == kBF16) launch_pool_flat_bwd_t<bf16_t>(dflat, flat, relu, arg, dx, B, k, p, bands, lb, s);
    else launch_pool_flat_bwd_t<float>(dflat, flat, relu, arg, dx, B, k, p, bands, lb, s);
    return launch_ok();
}

// ---------------------------------------------------------------- local response normalisation (across channels)
// One thread owns V consecutive channels (16 bytes) of one pixel and reads the channels up to 8 to either side
// (padding channels hold zeros, channels outside the tensor count as zeros), so windows of up to 9 channels fit
// the forward pass and the backward pass, which needs the window sums of the neighbours' windows.
template <typename T> struct LrnWindow {
    static constexpr int V = 16 / sizeof(T), R = 8, N = V + 2 * R;
    float f[N];   // f[R + e] is channel c0 + e
    __device__ __forceinline__ void load(const T *pix, int c0, int Cp)
    {
#pragma unroll
        for (int q = -(R / V); q <= R / V; ++q) {
            const int c = c0 + q * V;
            Vec16<T> v;
            if (c >= 0 && c < Cp) v.u = *reinterpret_cast<const uint4 *>(pix + c);
            else v.u = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int e = 0; e < V; ++e) f[R + q * V + e] = ldf(&v.e[e]);
        }
    }
};
// s^(-e) for s >= bias > 0, far from the denormal range on both sides: the bare hardware log2 and exp2 (about one
// ulp each) without the range fix-ups of the library routines
__device__ __forceinline__ float pow_neg(float s, float e) { return __builtin_amdgcn_exp2f(-e * __builtin_amdgcn_logf(s)); }

template <typename T, int half>   // half = size / 2, a compile-time constant so that the windows stay in registers
__global__ __launch_bounds__(256) void lrn_fwd_kernel(const T *__restrict__ a, T *__restrict__ y, size_t groups, int Cp, float alpha, float beta,
                                                    float bias)
{
    constexpr int V = LrnWindow<T>::V, R = LrnWindow<T>::R;
    const size_t g = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= groups) return;
    const int cv = Cp / V;
    const size_t pix = g / cv;
    const int c0 = (int)(g - pix * cv) * V;
    LrnWindow<T> w;
    w.load(a + pix * Cp, c0, Cp);
    Vec16<T> o;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        float sum = 0.f;
#pragma unroll
        for (int j = -half; j <= half; ++j) sum += w.f[R + e + j] * w.f[R + e + j];
        stf(&o.e[e], w.f[R + e] * pow_neg(bias + alpha * sum, beta));
    }
    *reinterpret_cast<uint4 *>(y + pix * Cp + c0) = o.u;
}

template <typename T, int half>
__global__ __launch_bounds__(256) void lrn_bwd_kernel(const T *__restrict__ a, const T *__restrict__ dy, int relu, T *__restrict__ da, size_t groups,
                                                    int Cp, float alpha, float beta, float bias)
{
    constexpr int V = LrnWindow<T>::V, R = LrnWindow<T>::R;
    const size_t g = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= groups) return;
    const int cv = Cp / V;
    const size_t pix = g / cv;
    const int c0 = (int)(g - pix * cv) * V;
    LrnWindow<T> wa, wd;
    wa.load(a + pix * Cp, c0, Cp);
    wd.load(dy + pix * Cp, c0, Cp);
    // for every channel j within `half` of this thread's channels: s_j, and t_j = dy_j * a_j * s_j^(-beta-1)
    float t[V + 8], pown[V];   // pown: s^(-beta) of the thread's own channels
#pragma unroll
    for (int q = 0; q < V + 8; ++q) {
        const int j = q - 4;                    // channel c0 + j, j in [-4, V+3] covers half <= 4
        t[q] = 0.f;
        if (j >= -half && j < V + half) {       // decided at compile time
            float sum = 0.f;
#pragma unroll
            for (int r = -half; r <= half; ++r) sum += wa.f[R + j + r] * wa.f[R + j + r];
            const float sj = bias + alpha * sum;
            float pj1;                          // s^(-beta-1)
            if (j >= 0 && j < V) {              // own channel: s^(-beta) is needed too, one reciprocal gives the other
                pown[j] = pow_neg(sj, beta);
                pj1 = pown[j] * __builtin_amdgcn_rcpf(sj);
            } else {
                pj1 = pow_neg(sj, beta + 1.f);
            }
            t[q] = wd.f[R + j] * wa.f[R + j] * pj1;
        }
    }
    Vec16<T> o;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        float acc = 0.f;
#pragma unroll
        for (int r = -half; r <= half; ++r) acc += t[e + 4 + r];
        float v = wd.f[R + e] * pown[e] - 2.f * alpha * beta * wa.f[R + e] * acc;
        if (relu && !(wa.f[R + e] > 0.f)) v = 0.f;
        stf(&o.e[e], v);
    }
    *reinterpret_cast<uint4 *>(da + pix * Cp + c0) = o.u;
}

template <typename T, int HALF>
static void launch_lrn_t(const void *a, const void *dy, int relu, void *out, size_t groups, int Cp, float alpha, float beta, float bias, bool bwd,
                         hipStream_t s)
{
    const unsigned blocks = blocks_for(groups, 256);
    if (bwd)
        hipLaunchKernelGGL((lrn_bwd_kernel<T, HALF>), dim3(blocks), dim3(256), 0, s, static_cast<const T *>(a), static_cast<const T *>(dy), relu,
                           static_cast<T *>(out), groups, Cp, alpha, beta, bias);
    else
        hipLaunchKernelGGL((lrn_fwd_kernel<T, HALF>), dim3(blocks), dim3(256), 0, s, static_cast<const T *>(a), static_cast<T *>(out), groups, Cp, alpha,
                           beta, bias);
}
template <typename T>
static int launch_lrn_any(const void *a, const void *dy, int relu, void *out, size_t pixels, int Cp, int size, float alpha, float beta, float bias,
                          bool bwd, hipStream_t s)
{
    if (size < 1 || size > 9 || !(size & 1) || !(bias > 0.f)) return -1;
    const size_t groups = pixels * (size_t)(Cp / (16 / (int)sizeof(T)));
    switch (size / 2) {
    case 0: launch_lrn_t<T, 0>(a, dy, relu, out, groups, Cp, alpha, beta, bias, bwd, s); break;
    case 1: launch_lrn_t<T, 1>(a, dy, relu, out, groups, Cp, alpha, beta, bias, bwd, s); break;
    case 2: launch_lrn_t<T, 2>(a, dy, relu, out, groups, Cp, alpha, beta, bias, bwd, s); break;
    case 3: launch_lrn_t<T, 3>(a, dy, relu, out, groups, Cp, alpha, beta, bias, bwd, s); break;
    default: launch_lrn_t<T, 4>(a, dy, relu, out, groups, Cp, alpha, beta, bias, bwd, s); break;
    }
    return launch_ok();
}
int launch_lrn_fwd(int dtype, const void *a, void *y, size_t pixels, int Cp, int size, float alpha, float beta, float bias, hipStream_t s)
{
    return dtype == kBF16 ? launch_lrn_any<bf16_t>(a, nullptr, 0, y, pixels, Cp, size, alpha, beta, bias, false, s)
                          : launch_lrn_any<float>(a, nullptr, 0, y, pixels, Cp, size, alpha, beta, bias, false, s);
}
int launch_lrn_bwd(int dtype, const void *a, const void *dy, int relu, void *da, size_t pixels, int Cp, int size, float alpha, float beta,
                   float bias, hipStream_t s)
{
    return dtype == kBF16 ? launch_lrn_any<bf16_t>(a, dy, relu, da, pixels, Cp, size, alpha, beta, bias, true, s)
                          : launch_lrn_any<float>(a, dy, relu, da, pixels, Cp, size, alpha, beta, bias, true, s);
}

// ---------------------------------------------------------------- response normalisation and the pool on top of it, in one pass
// The normalised tensor is as large as the convolution's output and nothing but the pool reads it; the gradient at the pool's
// input nothing but the normalisation's backward pass.  Both stay in LDS here, rounded to the element type where the separate
// kernels store them.  Bound by the vector units (two or three transcendentals and about 25 other instructions per
// element) a little above HBM's time.  bf16, 128 images, separate kernels / here: 96 channels 55 x 55 forward 52 / 33 us, backward with
// the first stage of the bias gradient 110 / 59; 256 channels 27 x 27 forward 37 / 21, backward 75 / 45.
// Channels c0 - S .. c0 + V + S - 1 of a pixel around the V channels of a thread; channels outside the tensor count as zeros.
template <typename T, int S> struct LrnNear {
    static constexpr int V = 16 / sizeof(T);
    float f[V + 2 * S];   // f[S + e] is channel c0 + e
    struct alignas(4 * sizeof(T)) Four { T e[4]; };
    __device__ __forceinline__ void load(const T *pix, int c0, int Cp)
    {
        Vec16<T> v;
        v.u = *reinterpret_cast<const uint4 *>(pix + c0);
        Four l[S / 4], r[S / 4];
#pragma unroll
        for (int q = 0; q < S / 4; ++q) {
            l[q] = Four{}; r[q] = Four{};
            if (c0 - S + 4 * q >= 0) l[q] = *reinterpret_cast<const Four *>(pix + c0 - S + 4 * q);
            if (c0 + V + 4 * q < Cp) r[q] = *reinterpret_cast<const Four *>(pix + c0 + V + 4 * q);
        }
#pragma unroll
        for (int e = 0; e < V; ++e) f[S + e] = ldf(&v.e[e]);
#pragma unroll
        for (int e = 0; e < S; ++e) { f[e] = ldf(&l[e / 4].e[e % 4]); f[S + V + e] = ldf(&r[e / 4].e[e % 4]); }
    }
};

// Forward.  A block makes R pooled rows of one image for `groups` channel groups of 16 bytes: it normalises the rows its windows
// touch once into LDS (2R + K - 2 of them; the one that two blocks share is done twice), then pools out of LDS.
struct LrnPool {
    int H, W, Cp, Ho, Wo, cv;              // cv: channel groups of a pixel
    int groups, R, tiles, chunks, cols;    // forward: groups per block, pooled rows per block, blocks per image (rows, groups), input columns used
    int lanes, wlanes, Hb, Wb;             // backward: pixels side by side in a block and in a wavefront, 2 x 2 blocks of input pixels
    FastDiv dgroups, dtiles, dchunks, dcols, dWo, dcv, dHb;
    float alpha, beta, bias;
};
constexpr int kLrnPoolLds = 40 << 10;      // forward: four blocks a CU
template <typename T, int HALF, int K>
__global__ __launch_bounds__(256) void lrn_pool_fwd_kernel(const T *__restrict__ a, T *__restrict__ y, uint8_t *__restrict__ arg, LrnPool p)
{
    constexpr int V = Vec16<T>::N, S = 4;
    extern __shared__ uint4 tile[];
    uint32_t t = xcd_block();
    uint32_t q = fdiv32(t, p.dchunks);
    const int g0 = (int)(t - q * p.chunks) * p.groups;
    t = q; q = fdiv32(t, p.dtiles);
    const int py0 = (int)(t - q * p.tiles) * p.R, n = (int)q;
    const int rows_out = min(p.R, p.Ho - py0), rows_in = 2 * (rows_out - 1) + K;
    const T *src = a + ((long)n * p.H + 2 * py0) * p.W * p.Cp;
    const int pieces = rows_in * p.cols * p.groups;
    // two pieces of a thread in flight
    for (int i = threadIdx.x; i < pieces; i += 512) {
        LrnNear<T, S> w[2];
        bool ok[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = i + u * 256;
            const uint32_t pix = fdiv32((uint32_t)j, p.dgroups), row = fdiv32(pix, p.dcols);
            const int c0 = (g0 + j - (int)pix * p.groups) * V;
            ok[u] = j < pieces && c0 < p.Cp;
            if (ok[u]) w[u].load(src + ((long)row * p.W + (pix - row * p.cols)) * p.Cp, c0, p.Cp);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (!ok[u]) continue;
            Vec16<T> o;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                float sum = 0.f;
#pragma unroll
                for (int j = -HALF; j <= HALF; ++j) sum += w[u].f[S + e + j] * w[u].f[S + e + j];
                stf(&o.e[e], w[u].f[S + e] * pow_neg(p.bias + p.alpha * sum, p.beta));
            }
            tile[i + u * 256] = o.u;
        }
    }
    __syncthreads();
    const int outs = rows_out * p.Wo * p.groups;
    for (int i = threadIdx.x; i < outs; i += 256) {
        const uint32_t pix = fdiv32((uint32_t)i, p.dgroups), row = fdiv32(pix, p.dWo);
        const int g = i - (int)pix * p.groups, px = (int)(pix - row * p.Wo), c0 = (g0 + g) * V;
        if (c0 >= p.Cp) continue;
        Vec16<T> v[K * K];
#pragma unroll
        for (int j = 0; j < K * K; ++j) v[j].u = tile[((2 * (int)row + j / K) * p.cols + 2 * px + j % K) * p.groups + g];
        Vec16<T> o;
        uint64_t packed;
        first_max<T, K * K, sizeof(T) == 2>(v, o, packed);
        const long off = (((long)n * p.Ho + py0 + row) * p.Wo + px) * p.Cp + c0;
        *reinterpret_cast<uint4 *>(y + off) = o.u;
        if (V == 8) *reinterpret_cast<uint64_t *>(arg + off) = packed;
        else *reinterpret_cast<uint32_t *>(arg + off) = (uint32_t)packed;
    }
}

// the value of the lane before / after this one in the wavefront (anything at its ends)
__device__ __forceinline__ float lane_before(float v) { return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x138, 0xF, 0xF, true)); }
__device__ __forceinline__ float lane_after(float v) { return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x130, 0xF, 0xF, true)); }

// Backward.  A block makes two rows of the convolution's output gradient, all channels: the pool's gradient at them into LDS (as
// pool_bwd_s2_kernel forms it, a 2 x 2 block of pixels per thread), then the normalisation's, times [a > 0].  A wavefront
// holds whole pixels, 64 / cv of them, so that what a thread needs of its neighbours' channels comes from the lanes beside it,
// each power worked out once.  A thread keeps its channel group, so that it can also add up the columns of what it stores
// (bands[column][block], the first stage of that convolution's bias gradient).
template <typename T, int HALF, int K>
__global__ __launch_bounds__(256, 6) void lrn_pool_bwd_kernel(const T *__restrict__ a, const T *__restrict__ dy, const uint8_t *__restrict__ arg,
                                                         T *__restrict__ da, LrnPool p, float *__restrict__ bands)
{
    constexpr int V = Vec16<T>::N;
    extern __shared__ uint4 tile[];
    const uint32_t blk = xcd_block();
    const int n = (int)fdiv32(blk, p.dHb), jy = (int)blk - n * p.Hb;
    const int lane = threadIdx.x & 63, wl = (int)fdiv32((uint32_t)lane, p.dcv);   // pixel within the wavefront
    const int cg = lane - wl * p.cv, c0 = cg * V, pl = (int)(threadIdx.x >> 6) * p.wlanes + wl;
    const bool live = wl < p.wlanes;
    const int rows = min(2, p.H - 2 * jy);
    const size_t pooled = (size_t)p.Ho * p.Wo * p.Cp;   // of one image
    const __amdgpu_buffer_rsrc_t rdy = byte_range(dy + n * pooled, pooled * sizeof(T)), rarg = byte_range(arg + n * pooled, pooled);
    for (int jx = pl; live && jx < p.Wb; jx += p.lanes) {
        PoolWindows<T> win;
        win.load(rdy, rarg, (unsigned)(((jy - 1) * p.Wo + jx - 1) * p.Cp + c0), jy, jx, p.Ho, p.Wo, p.Cp);
        float acc[4][V];
        win.template sums<K>(acc);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int by = b >> 1, ix = 2 * jx + (b & 1);
            if (by < rows && ix < p.W) {
                Vec16<T> o;
#pragma unroll
                for (int e = 0; e < V; ++e) stf(&o.e[e], acc[b][e]);
                tile[(by * p.W + ix) * p.cv + cg] = o.u;
            }
        }
    }
    __syncthreads();
    float colsum[V];
#pragma unroll
    for (int e = 0; e < V; ++e) colsum[e] = 0.f;
    const long base = ((long)n * p.H + 2 * jy) * p.W * p.Cp + c0;
    const int npix = rows * p.W;
    const bool first = cg == 0, last = cg == p.cv - 1;
    // channels up to HALF away sit in the next lane, or (four channels a lane, HALF never more than 4) there too
    static_assert(HALF <= V, "a window reaches no further than the neighbouring lanes");
    for (int i = pl; live && i < npix; i += p.lanes) {
        Vec16<T> av, dv;
        av.u = *reinterpret_cast<const uint4 *>(a + base + (long)i * p.Cp);
        dv.u = tile[i * p.cv + cg];
        float f[V + 2 * HALF], t[V + 2 * HALF], pown[V];   // [HALF + e] is channel c0 + e; t: dy * a * s^(-beta-1); pown: s^(-beta)
#pragma unroll
        for (int e = 0; e < V; ++e) f[HALF + e] = ldf(&av.e[e]);
#pragma unroll
        for (int e = 0; e < HALF; ++e) {
            const float l = lane_before(f[V + e]), r = lane_after(f[HALF + e]);
            f[e] = first ? 0.f : l;
            f[HALF + V + e] = last ? 0.f : r;
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r <= 2 * HALF; ++r) sum += f[e + r] * f[e + r];
            const float s = p.bias + p.alpha * sum;
            pown[e] = pow_neg(s, p.beta);
            t[HALF + e] = ldf(&dv.e[e]) * f[HALF + e] * (pown[e] * __builtin_amdgcn_rcpf(s));
        }
#pragma unroll
        for (int e = 0; e < HALF; ++e) {
            const float l = lane_before(t[V + e]), r = lane_after(t[HALF + e]);
            t[e] = first ? 0.f : l;
            t[HALF + V + e] = last ? 0.f : r;
        }
        Vec16<T> o;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float acc = 0.f;
#pragma unroll
            for (int r = 0; r <= 2 * HALF; ++r) acc += t[e + r];
            float v = ldf(&dv.e[e]) * pown[e] - 2.f * p.alpha * p.beta * f[HALF + e] * acc;
            if (!(f[HALF + e] > 0.f)) v = 0.f;
            stf(&o.e[e], v);
            colsum[e] += ldf(&o.e[e]);
        }
        *reinterpret_cast<uint4 *>(da + base + (long)i * p.Cp) = o.u;
    }
    __syncthreads();
    float *part = reinterpret_cast<float *>(tile);   // [lane][channel]
    if (live) {
#pragma unroll
        for (int e = 0; e < V; ++e) part[pl * p.Cp + c0 + e] = colsum[e];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < p.Cp; c += 256) {
        float s = 0.f;
        for (int j = 0; j < p.lanes; ++j) s += part[j * p.Cp + c];
        bands[(long)c * gridDim.x + blk] = s;
    }
}

// Where the pair runs as one kernel: pools of 2 or 3 with stride 2, rows that fit LDS, pixels that fit a wavefront.
static bool lrn_pool_plan(int dtype, int B, int H, int W, int Cp, int k, int stride, LrnPool &p, size_t &lds_fwd, size_t &lds_bwd)
{
    const int V = dtype == kBF16 ? 8 : 4;
    if (!pool_bwd_blocks(H, W, Cp, (int)dtype_size(dtype), k, stride) || H < k || W < k) return false;
    p.H = H; p.W = W; p.Cp = Cp; p.Ho = (H - k) / 2 + 1; p.Wo = (W - k) / 2 + 1; p.cv = Cp / V;
    if (p.cv > 64) return false;
    p.cols = 2 * (p.Wo - 1) + k;
    // 64 bytes of a pixel per block: fewer re-read the row that two blocks share less often, more leave room for fewer rows
    p.groups = p.cv < 4 ? p.cv : 4;
    p.chunks = (p.cv + p.groups - 1) / p.groups;
    const long row = (long)p.cols * p.groups * 16;
    const long fit = (kLrnPoolLds / row - k) / 2 + 1;   // pooled rows whose input rows fit
    if (kLrnPoolLds / row < k) return false;
    // and fewer while CUs are idle and a block would take more than one round of its threads (bf16, 55 x 55 over 96 channels, 1 image: a
    // pass 115 us with 6 blocks for the rows, 110 with 27; fp32, 8 x 11 over 64, 3 images, one round: 92.9 in 1, 94.3 in 3)
    const long round = std::max(1L, (512 / ((long)p.cols * p.groups) - k) / 2 + 1);
    p.tiles = (int)std::max((p.Ho + fit - 1) / fit, std::min((p.Ho + round - 1) / round, 256 / ((long)B * p.chunks)));
    p.R = (p.Ho + p.tiles - 1) / p.tiles;
    p.tiles = (p.Ho + p.R - 1) / p.R;
    lds_fwd = (size_t)(2 * (p.R - 1) + k) * (size_t)row;
    p.wlanes = 64 / p.cv; p.lanes = 4 * p.wlanes; p.Hb = (H + 1) / 2; p.Wb = (W + 1) / 2;
    const long tile = 2l * W * p.cv * 16, sums = (long)p.lanes * Cp * 4;
    if (tile > (64 << 10)) return false;
    lds_bwd = (size_t)(tile > sums ? tile : sums);
    p.dgroups = make_fastdiv(p.groups); p.dtiles = make_fastdiv(p.tiles); p.dchunks = make_fastdiv(p.chunks); p.dcols = make_fastdiv(p.cols);
    p.dWo = make_fastdiv(p.Wo); p.dcv = make_fastdiv(p.cv); p.dHb = make_fastdiv(p.Hb);
    return true;
}
long lrn_pool_bands(int dtype, int B, int H, int W, int Cp, int k, int stride, bool forked, bool always)
{
    LrnPool p;
    size_t f, b;
    if (!lrn_pool_plan(dtype, B, H, W, Cp, k, stride, p, f, b)) return 0;
    const long blocks = (long)B * p.Hb;
    if ((long)B * p.tiles * p.chunks > 0x7fffffffL || blocks > 0x7fffffffL) return 0;
    // A block of the backward kernel takes 2 * W pixels, p.lanes side by side, in up to 18 rounds: in bf16 more than nine of them on
    // less than a quarter of the CUs are longer than the launches and the tensors they save, unless there is hardly anything to do.  A
    // pass of two convolutions, separate / here, us: 55 x 55 over 256 channels (14 rounds) 1 image 108 / 118, 2 images (56 blocks)
    // 116 / 120, 4 images (112) 130 / 126; 17 x 84 over 128 (10.5 rounds) 3 images (27 blocks) 107 / 112; 16 x 85 over 128 1 image (8
    // blocks) 101 / 95; 19 x 23 over 256 (6 rounds) 3 images 98 / 88; fp32 25 x 88 over 64 (11 rounds) 1 image 103 / 105, 36 x 22 over
    // 256 (11 rounds) 114 / 108.  With the side stream the separate kernels are never ahead: AlexNet-style net with two normalised
    // layers, 1 image, 424 / 417.  Over 58 passes without and 82 with it the choice is at most 1.02 of the better one.
    if (!always && !forked && dtype == kBF16 && 2 * W > 9 * p.lanes && blocks >= 20 && blocks < 60) return 0;
    return blocks;
}
template <typename T, int HALF>
static void launch_lrn_pool_t(const LrnPool &p, int B, int k, size_t lds, const void *a, void *y, const void *dy, uint8_t *arg, void *da, float *bands,
                              hipStream_t s)
{
    const T *aa = static_cast<const T *>(a);
    if (da) {
        const dim3 grid((unsigned)(B * p.Hb));
        const T *g = static_cast<const T *>(dy);
        T *o = static_cast<T *>(da);
        if (k == 3) hipLaunchKernelGGL((lrn_pool_bwd_kernel<T, HALF, 3>), grid, dim3(256), lds, s, aa, g, arg, o, p, bands);
        else hipLaunchKernelGGL((lrn_pool_bwd_kernel<T, HALF, 2>), grid, dim3(256), lds, s, aa, g, arg, o, p, bands);
    } else {
        const dim3 grid((unsigned)(B * p.tiles * p.chunks));
        if (k == 3) hipLaunchKernelGGL((lrn_pool_fwd_kernel<T, HALF, 3>), grid, dim3(256), lds, s, aa, static_cast<T *>(y), arg, p);
        else hipLaunchKernelGGL((lrn_pool_fwd_kernel<T, HALF, 2>), grid, dim3(256), lds, s, aa, static_cast<T *>(y), arg, p);
    }
}
template <typename T>
static int launch_lrn_pool(int dtype, int B, int H, int W, int Cp, int size, float alpha, float beta, float bias, int k, const void *a, void *y,
                           const void *dy, const uint8_t *arg, void *da, float *bands, hipStream_t s)
{
    LrnPool p;
    size_t lf, lb;
    if (size < 1 || size > 9 || !(size & 1) || !(bias > 0.f)) return -1;
    if (lrn_pool_bands(dtype, B, H, W, Cp, k, 2, false, true) == 0 || !lrn_pool_plan(dtype, B, H, W, Cp, k, 2, p, lf, lb)) return -1;
    p.alpha = alpha; p.beta = beta; p.bias = bias;
    const size_t lds = da ? lb : lf;
    uint8_t *ar = const_cast<uint8_t *>(arg);
    switch (size / 2) {
    case 0: launch_lrn_pool_t<T, 0>(p, B, k, lds, a, y, dy, ar, da, bands, s); break;
    case 1: launch_lrn_pool_t<T, 1>(p, B, k, lds, a, y, dy, ar, da, bands, s); break;
    case 2: launch_lrn_pool_t<T, 2>(p, B, k, lds, a, y, dy, ar, da, bands, s); break;
    case 3: launch_lrn_pool_t<T, 3>(p, B, k, lds, a, y, dy, ar, da, bands, s); break;
    default: launch_lrn_pool_t<T, 4>(p, B, k, lds, a, y, dy, ar, da, bands, s); break;
    }
    return launch_ok();
}
int launch_lrn_pool_fwd(int dtype, const void *a, void *y, uint8_t *arg, int B, int H, int W, int Cp, int size, float alpha, float beta, float bias, int k,
                        hipStream_t s)
{
    return dtype == kBF16 ? launch_lrn_pool<bf16_t>(dtype, B, H, W, Cp, size, alpha, beta, bias, k, a, y, nullptr, arg, nullptr, nullptr, s)
                          : launch_lrn_pool<float>(dtype, B, H, W, Cp, size, alpha, beta, bias, k, a, y, nullptr, arg, nullptr, nullptr, s);
}
int launch_lrn_pool_bwd(int dtype, const void *a, const void *dy, const uint8_t *arg, void *da, int B, int H, int W, int Cp, int size, float alpha,
                        float beta, float bias, int k, float *bands, hipStream_t s)
{
    return dtype == kBF16 ? launch_lrn_pool<bf16_t>(dtype, B, H, W, Cp, size, alpha, beta, bias, k, a, nullptr, dy, arg, da, bands, s)
                          : launch_lrn_pool<float>(dtype, B, H, W, Cp, size, alpha, beta, bias, k, a, nullptr, dy, arg, da, bands, s);
}

// ---------------------------------------------------------------- flatten / unflatten
template <typename T>
__global__ __launch_bounds__(256) void flatten_kernel(const T *__restrict__ x, T *__restrict__ flat, int B, int H, int W, int C, int Cp)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;  // (b, c, h, w)
    if (i >= (long)B * C * H * W) return;
    const int w = (int)(i % W); long t = i / W;
    const int h = (int)(t % H); t /= H;
    const int c = (int)(t % C);
    const int b = (int)(t / C);
    flat[i] = x[(((long)b * H + h) * W + w) * Cp + c];
}
int launch_flatten(int dtype, const void *x, void *flat, int B, int H, int W, int C, int Cp, hipStream_t s)
{
    const unsigned blocks = blocks_for((size_t)B * C * H * W, 256);
    if (dtype == kBF16)
        hipLaunchKernelGGL(flatten_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, static_cast<const bf16_t *>(x), static_cast<bf16_t *>(flat), B, H, W, C, Cp);
    else
        hipLaunchKernelGGL(flatten_kernel<float>, dim3(blocks), dim3(256), 0, s, static_cast<const float *>(x), static_cast<float *>(flat), B, H, W, C, Cp);
    return launch_ok();
}

template <typename T>
__global__ __launch_bounds__(256) void unflatten_kernel(const T *__restrict__ dflat, const T *__restrict__ x, int relu, T *__restrict__ dx, int B, int H,
                                                      int W, int C, int Cp)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;  // (b, h, w, cp)
    if (i >= (long)B * H * W * Cp) return;
    const int c = (int)(i % Cp); long t = i / Cp;
    const int w = (int)(t % W); t /= W;
    const int h = (int)(t % H);
    const int b = (int)(t / H);
    float v = 0.f;
    if (c < C) {
        v = ldf(&dflat[(((long)b * C + c) * H + h) * W + w]);
        if (relu && !(ldf(&x[i]) > 0.f)) v = 0.f;
    }
    stf(&dx[i], v);
}
int launch_unflatten(int dtype, const void *dflat, const void *x, int relu, void *dx, int B, int H, int W, int C, int Cp, hipStream_t s)
{
    const unsigned blocks = blocks_for((size_t)B * H * W * Cp, 256);
    if (dtype == kBF16)
        hipLaunchKernelGGL(unflatten_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, static_cast<const bf16_t *>(dflat), static_cast<const bf16_t *>(x), relu,
                           static_cast<bf16_t *>(dx), B, H, W, C, Cp);
    else
        hipLaunchKernelGGL(unflatten_kernel<float>, dim3(blocks), dim3(256), 0, s, static_cast<const float *>(dflat), static_cast<const float *>(x), relu,
                           static_cast<float *>(dx), B, H, W, C, Cp);
    return launch_ok();
}

// ---------------------------------------------------------------- bias gradient (column sums)
// Stage 1: a block owns a band of rows and up to 256 column chunks of 16 bytes;
// thread (c, r) adds rows r, r+RL, ... of chunk c, the RL row lanes are then
// added in lane order.  Stage 2 adds the bands in a fixed tree.  No atomics, so
// the result does not depend on scheduling.
// Stage 1 for several tensors in one launch: a block finds its job and its (column group, band) in it.
template <typename T>
__global__ __launch_bounds__(256) void colsum_stage1(ColsumS1Jobs jobs)
{
    constexpr int V = 16 / sizeof(T);
    __shared__ float part[256 * V];
    int q = 0;
#pragma unroll
    for (int i = 1; i < 12; ++i) q += blockIdx.x >= jobs.j[i].start_block;
    const ColsumS1Job &J = jobs.j[q];
    const unsigned lb = blockIdx.x - J.start_block, bx = lb % (unsigned)J.gx, by = lb / (unsigned)J.gx;
    const T *dy = static_cast<const T *>(J.dy);
    const long ld = J.ld, M = J.M, rows_per_block = J.rows_per_block;
    const int chunks = J.chunks, cpb = J.cpb, rl = J.rl;
    const int c = threadIdx.x % cpb, r = threadIdx.x / cpb;
    const int gc = (int)bx * cpb + c;
    const long m0 = (long)by * rows_per_block, m1 = min(M, m0 + rows_per_block);
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (r < rl && gc < chunks) {
        union Vec { uint4 u; T e[V]; };
        const T *src = dy + (long)gc * V;
        long m = m0 + r;
        for (; m + 3 * rl < m1; m += 4 * rl) {   // four rows in flight, added in their order: fp32 128 images 21.0 -> 17.7 us, bf16 256 images 23.7 -> 21.4
            Vec v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u].u = *reinterpret_cast<const uint4 *>(src + (m + u * rl) * ld);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) acc[e] += ldf(&v[u].e[e]);
        }
        for (; m < m1; m += rl) {
            Vec v;
            v.u = *reinterpret_cast<const uint4 *>(src + m * ld);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] += ldf(&v.e[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) part[threadIdx.x * V + e] = acc[e];
    __syncthreads();
    if (r == 0 && gc < chunks) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float t = 0.f;
            for (int j = 0; j < rl; ++j) t += part[(j * cpb + c) * V + e];
            J.ws[(long)by * ld + (long)gc * V + e] = t;
        }
    }
}
// Stage 2 for several layers in one launch.
__device__ __forceinline__ void colsum_finish_block(const ColsumJobs &jobs, unsigned block, float (&part)[4][8])
{
    // Band-major jobs (ws[band][ld], from colsum_stage1, or the rows of a short tensor itself, up to 512 bands): 8 columns per block,
    // 32 lanes per column.
    // Column-major jobs (ws[column][nblk], from the pooling backward pass, thousands of bands): a block per column.  A
    // lane adds bands lane, lane + L, ... (eight loads in flight); the lanes are then added in a fixed tree, the lanes of
    // a wavefront by shuffles and its four wavefronts in LDS.  Latency bounds it: with a wavefront per column and one lane
    // adding the 32 or 64 partial sums from LDS, the AlexNet-style layers took 10.8 us at 128 images (bf16; now 7.7), 18.3 at
    // 256 (9.6), 17.8 in fp32 at 128 (9.2).
    int q = 0;
#pragma unroll
    for (int i = 1; i < 12; ++i) q += block >= jobs.j[i].start_block;   // independent scalar loads, no chain of them
    const ColsumJob &J = jobs.j[q];
    const float *ws = J.ws;
    const int nblk = J.nblk, N = J.N, cm = J.colmajor, cpb = cm ? 1 : 8, L = 256 / cpb;
    const int tx = cm ? 0 : threadIdx.x % 8, ty = cm ? threadIdx.x : threadIdx.x / 8;
    const int n = (int)(block - J.start_block) * cpb + tx;
    const long sb = cm ? 1 : J.ld, sn = cm ? nblk : 1;   // strides of the band and of the column index
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (n < N) {
        const float *col = ws + (long)n * sn;
        const bf16_t *half = reinterpret_cast<const bf16_t *>(ws) + (long)n * sn;
        int b = ty;
        for (; b + 7 * L < nblk; b += 8 * L) {
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] += J.bf16 ? (float)half[(long)(b + u * L) * sb] : col[(long)(b + u * L) * sb];
        }
#pragma unroll
        for (int u = 0; u < 7; ++u)
            if (b + u * L < nblk) a[u] += J.bf16 ? (float)half[(long)(b + u * L) * sb] : col[(long)(b + u * L) * sb];
    }
    float t = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    for (int o = 32; o >= 8; o >>= 1) t += __shfl_xor(t, o, 64);   // lanes 8 apart hold the same band-major column
    if (cm) for (int o = 4; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (threadIdx.x % 64 < 8) part[threadIdx.x / 64][threadIdx.x % 64] = t;
    __syncthreads();
    if (ty == 0 && n < N) J.db[n] = ((part[0][tx] + part[1][tx]) + (part[2][tx] + part[3][tx])) / J.div;
}
__global__ __launch_bounds__(256) void colsum_stage2(ColsumJobs jobs)
{
    __shared__ float part[4][8];
    colsum_finish_block(jobs, blockIdx.x, part);
}
// The same with a reduction of partial sums (its first red.blocks workgroups).
template <typename T> __global__ __launch_bounds__(256) void colsum_stage2_reduce(ColsumJobs jobs, Reduction red)
{
    __shared__ ReduceShared sh;
    if (blockIdx.x < red.blocks) reduce_block<T>(red, blockIdx.x, sh);
    else colsum_finish_block(jobs, blockIdx.x - red.blocks, sh.part);
}
static void colsum_geometry(int dtype, long ld, long M, int &chunks, int &cpb, int &rl, long &rows_per_block, int &nblk)
{
    const int V = dtype == kBF16 ? 8 : 4;
    chunks = (int)(ld / V);
    cpb = chunks < 256 ? chunks : 256;
    rl = 256 / cpb;
    rows_per_block = (M + 511) / 512;
    if (rows_per_block < 4L * rl) rows_per_block = 4L * rl;
    rows_per_block = (rows_per_block + rl - 1) / rl * rl;
    nblk = (int)((M + rows_per_block - 1) / rows_per_block);
}
// Rows up to which the second stage takes the tensor itself (as many as there are bands at most): a first stage for the
// fully-connected layers alone costs a launch of 6 us in fp32 and 14 in bf16, where two blocks add up 93 rows.
constexpr long kColsumDirect = 512;
size_t colsum_ws_floats(int dtype, long M, long ld)
{
    if (M <= kColsumDirect) return 0;
    int chunks, cpb, rl, nblk; long rpb;
    colsum_geometry(dtype, ld, M, chunks, cpb, rl, rpb, nblk);
    return (size_t)nblk * (size_t)ld;
}
// dy is [M][ld] with ld a multiple of 8 and columns N..ld-1 zero or ignorable.  Stage 1 leaves the band sums in
// ws (colsum_ws_floats) and appends the job that finishes them; launch_colsum_finish runs all appended jobs.
int colsum_partial_defer(int dtype, const void *dy, long ld, long M, int N, float *db, float *ws, ColsumS1Jobs &s1, ColsumJobs &jobs)
{
    if (jobs.n >= 12 || s1.n >= 12 || (ld & 7) || M <= 0) return -1;
    if (M <= kColsumDirect) {
        ColsumJob &J = jobs.j[jobs.n++];
        J.ws = static_cast<const float *>(dy); J.nblk = (int)M; J.ld = ld; J.N = N; J.db = db;
        J.start_block = 0; J.colmajor = 0; J.bf16 = dtype == kBF16; J.div = 1.f;
        return 0;
    }
    int chunks, cpb, rl, nblk; long rpb;
    colsum_geometry(dtype, ld, M, chunks, cpb, rl, rpb, nblk);
    ColsumS1Job &S = s1.j[s1.n++];
    S.dy = dy; S.ws = ws; S.ld = ld; S.M = M; S.rows_per_block = rpb; S.chunks = chunks; S.cpb = cpb; S.rl = rl;
    S.gx = (chunks + cpb - 1) / cpb; S.gy = nblk; S.start_block = 0;
    ColsumJob &J = jobs.j[jobs.n++];
    J.ws = ws; J.nblk = nblk; J.ld = ld; J.N = N; J.db = db; J.start_block = 0; J.colmajor = 0; J.bf16 = 0; J.div = 1.f;
    return 0;
}
int launch_colsum_stage1(int dtype, ColsumS1Jobs &s1, hipStream_t s)
{
    if (s1.n == 0) return 0;
    unsigned long blocks = 0;
    for (int q = 0; q < s1.n; ++q) { s1.j[q].start_block = (unsigned)blocks; blocks += (unsigned long)s1.j[q].gx * (unsigned long)s1.j[q].gy; }
    if (blocks > 0x7fffffffu) return -1;
    for (int q = s1.n; q < 12; ++q) s1.j[q].start_block = ~0u;
    if (dtype == kBF16) hipLaunchKernelGGL(colsum_stage1<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, s, s1);
    else hipLaunchKernelGGL(colsum_stage1<float>, dim3((unsigned)blocks), dim3(256), 0, s, s1);
    s1.n = 0;
    return launch_ok();
}
int launch_colsum_partial(int dtype, const void *dy, long ld, long M, int N, float *db, float *ws, ColsumJobs &jobs, hipStream_t s)
{
    ColsumS1Jobs s1; s1.n = 0;
    if (colsum_partial_defer(dtype, dy, ld, M, N, db, ws, s1, jobs) != 0) return -1;
    return launch_colsum_stage1(dtype, s1, s);
}
int launch_colsum_finish(int dtype, ColsumJobs &jobs, const Reduction *beside, hipStream_t s)
{
    if (jobs.n == 0) return beside ? launch_reduction(dtype, *beside, s) : 0;
    unsigned blocks = 0;
    for (int q = 0; q < jobs.n; ++q) {
        ColsumJob &J = jobs.j[q];
        const int cpb = J.colmajor ? 1 : 8;
        J.start_block = blocks;
        blocks += (unsigned)((J.N + cpb - 1) / cpb);
    }
    for (int q = jobs.n; q < 12; ++q) jobs.j[q].start_block = ~0u;
    if (!beside) hipLaunchKernelGGL(colsum_stage2, dim3(blocks), dim3(256), 0, s, jobs);
    else if (dtype == kBF16) hipLaunchKernelGGL(colsum_stage2_reduce<bf16_t>, dim3(blocks + beside->blocks), dim3(256), 0, s, jobs, *beside);
    else hipLaunchKernelGGL(colsum_stage2_reduce<float>, dim3(blocks + beside->blocks), dim3(256), 0, s, jobs, *beside);
    jobs.n = 0;
    return launch_ok();
}

// ---------------------------------------------------------------- softmax cross-entropy
// One workgroup per row: lse = max + log(sum exp(z - max)); the row's loss is
// lse - z[label]; dz = (exp(z - lse) - [c == label]) / B.
__device__ inline float wave_max(float v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline float wave_sum(float v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// One workgroup per row: the four wavefronts each reduce their part, the four results meet in LDS.
__device__ inline float block_max(float v, float *sh)
{
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    v = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
    __syncthreads();
    return v;
}
__device__ inline float block_sum(float v, float *sh)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    v = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
    return v;
}
template <typename T>
__global__ __launch_bounds__(256) void softmax_ce_kernel(const float *__restrict__ z, long ld, const int32_t *__restrict__ labels, int B, int C,
                                                       T *__restrict__ dz, float *__restrict__ row_loss)
{
    __shared__ float sh[4];
    const int row = blockIdx.x, t = threadIdx.x;
    const float *zr = z + (long)row * ld;
    // the first four strides of the row stay in registers (all of it up to 1024 classes)
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = t + u * 256 < C ? zr[t + u * 256] : -INFINITY;
    float m = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
    for (int c = t + 1024; c < C; c += 256) m = fmaxf(m, zr[c]);
    m = block_max(m, sh);
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) sum += t + u * 256 < C ? expf(v[u] - m) : 0.f;
    for (int c = t + 1024; c < C; c += 256) sum += expf(zr[c] - m);
    sum = block_sum(sum, sh);
    const float lse = m + logf(sum);
    const int label = labels[row];
    // a label outside [0, C) addresses nothing: the row's loss (and with it the mean) becomes NaN, and dz is
    // the plain softmax / B, since no class compares equal to it below
    const bool label_ok = (unsigned)label < (unsigned)C;
    if (t == 0) row_loss[row] = label_ok ? lse - zr[label] : __builtin_nanf("");
    const float inv_b = 1.f / (float)B;
    T *dr = dz + (long)row * ld;
    for (int c = t; c < (int)ld; c += 256) {
        float g = 0.f;
        if (c < C) {
            g = (expf(zr[c] - lse) - (c == label ? 1.f : 0.f)) * inv_b;
        }
        stf(&dr[c], g);
    }
}
int launch_softmax_ce(int dtype, const float *z, long ld, const int32_t *labels, int B, int C, void *dz, float *row_loss, hipStream_t s)
{
    const unsigned blocks = (unsigned)B;
    if (dtype == kBF16) hipLaunchKernelGGL(softmax_ce_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, z, ld, labels, B, C, static_cast<bf16_t *>(dz), row_loss);
    else hipLaunchKernelGGL(softmax_ce_kernel<float>, dim3(blocks), dim3(256), 0, s, z, ld, labels, B, C, static_cast<float *>(dz), row_loss);
    return launch_ok();
}

// The mean of the row losses is one column of B bands: the launch that finishes the bias gradients takes it along (a kernel
// of its own cost 4 us in the middle of every pass).
void loss_job(const float *row_loss, int B, float *loss, ColsumJobs &jobs)
{
    ColsumJob &J = jobs.j[jobs.n++];
    J.ws = row_loss; J.nblk = B; J.ld = 1; J.N = 1; J.db = loss; J.start_block = 0; J.colmajor = 1; J.bf16 = 0; J.div = (float)B;
}

// ---------------------------------------------------------------- debug exports
template <typename T>
__global__ __launch_bounds__(256) void export_nhwc_kernel(const T *__restrict__ x, float *__restrict__ dst, int B, int H, int W, int C, int Cp)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;  // (b, c, h, w)
    if (i >= (long)B * C * H * W) return;
    const int w = (int)(i % W); long t = i / W;
    const int h = (int)(t % H); t /= H;
    const int c = (int)(t % C);
    const int b = (int)(t / C);
    dst[i] = ldf(&x[(((long)b * H + h) * W + w) * Cp + c]);
}
int launch_export_nhwc(int dtype, const void *x, float *dst, int B, int H, int W, int C, int Cp, hipStream_t s)
{
    const unsigned blocks = blocks_for((size_t)B * C * H * W, 256);
    if (dtype == kBF16) hipLaunchKernelGGL(export_nhwc_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, static_cast<const bf16_t *>(x), dst, B, H, W, C, Cp);
    else hipLaunchKernelGGL(export_nhwc_kernel<float>, dim3(blocks), dim3(256), 0, s, static_cast<const float *>(x), dst, B, H, W, C, Cp);
    return launch_ok();
}
template <typename T> __global__ __launch_bounds__(256) void export_rows_kernel(const T *__restrict__ x, long ld, float *__restrict__ dst, int B, int F)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long)B * F) return;
    const long b = i / F, f = i - b * F;
    dst[i] = ldf(&x[b * ld + f]);
}
int launch_export_rows(int dtype, int src_f32, const void *x, long ld, float *dst, int B, int F, hipStream_t s)
{
    const unsigned blocks = blocks_for((size_t)B * F, 256);
    if (dtype == kBF16 && !src_f32) hipLaunchKernelGGL(export_rows_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, static_cast<const bf16_t *>(x), ld, dst, B, F);
    else hipLaunchKernelGGL(export_rows_kernel<float>, dim3(blocks), dim3(256), 0, s, static_cast<const float *>(x), ld, dst, B, F);
    return launch_ok();
}
__global__ __launch_bounds__(256) void export_argmax_kernel(const uint8_t *__restrict__ arg, uint8_t *__restrict__ dst, int B, int H, int W, int C, int Cp)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;  // (b, c, h, w)
    if (i >= (long)B * C * H * W) return;
    const int w = (int)(i % W); long t = i / W;
    const int h = (int)(t % H); t /= H;
    const int c = (int)(t % C);
    const int b = (int)(t / C);
    dst[i] = arg[(((long)b * H + h) * W + w) * Cp + c];
}
int launch_export_argmax(const uint8_t *arg, uint8_t *dst, int B, int H, int W, int C, int Cp, hipStream_t s)
{
    hipLaunchKernelGGL(export_argmax_kernel, dim3(blocks_for((size_t)B * C * H * W, 256)), dim3(256), 0, s, arg, dst, B, H, W, C, Cp);
    return launch_ok();
}
__global__ __launch_bounds__(256) void dropout_mask_kernel(uint8_t *dst, size_t count, uint64_t key, uint32_t thr)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const uint32_t u = (uint32_t)(mix64(key + 0x9E3779B97F4A7C15ull * (uint64_t)(i + 1)) >> 32);
    dst[i] = u >= thr ? 1 : 0;
}
int launch_dropout_mask(uint8_t *dst, size_t count, uint64_t key, uint32_t thr, hipStream_t s)
{
    hipLaunchKernelGGL(dropout_mask_kernel, dim3(blocks_for(count, 256)), dim3(256), 0, s, dst, count, key, thr);
    return launch_ok();
}

}  // namespace asgd
