// Partial sums of a split GEMM added up in a fixed order: device routines, each for one workgroup of up to 256 threads of a launch of its own or of
// a launch that does something else beside it (see Reduction in asgd_internal.h).
#pragma once
#include "asgd_internal.h"
#include "mfma_common.h"

namespace asgd {

template <typename T> __device__ __forceinline__ void reduce_plain(const float *ws, int splits, const Epilogue &ep, int M, int N, unsigned block)
{
    const long g = (long)block * 256 + threadIdx.x;
    const int n8 = N / 8;
    if (g >= (long)M * n8) return;
    const int m = (int)(g / n8), n0 = (int)(g - (long)m * n8) * 8;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const long stride = (long)M * N;
    const float *p0 = ws + (long)m * N + n0;
    int s = 0;
    for (; s + 4 <= splits; s += 4) {   // four partials in flight; added in split order all the same
        float4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float4 *p = reinterpret_cast<const float4 *>(p0 + (s + u) * stride);
            a[u] = p[0]; b[u] = p[1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[0] += a[u].x; v[1] += a[u].y; v[2] += a[u].z; v[3] += a[u].w;
            v[4] += b[u].x; v[5] += b[u].y; v[6] += b[u].z; v[7] += b[u].w;
        }
    }
    for (; s < splits; ++s) {
        const float4 *p = reinterpret_cast<const float4 *>(p0 + s * stride);
        const float4 a = p[0], b = p[1];
        v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w;
        v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
    }
    float b8[8];
    load_bias8<T>(ep, n0, b8);
    epilogue8<T>(ep, m, n0, v, b8);
}

// The same for few outputs and many partial sums (the first layer's filter gradient: 5280 groups of 8 outputs, up
// to 256 partials each): L = 8 or 32 neighbouring lanes, or with L = 256 a workgroup, share a group, lane l adds partials l, l+L,
// ... in that order, and the L sums are combined in a fixed butterfly (and the four wavefronts' in their order), so the
// result does not depend on anything but the inputs.
template <typename T, int L>
__device__ __forceinline__ void reduce_wide(const float *ws, int splits, const Epilogue &ep, int M, int N, unsigned block, float (&part)[4][8])
{
    static_assert(L == 8 || L == 32 || L == 256, "lanes per group of outputs");
    constexpr int SH = L == 8 ? 3 : L == 32 ? 5 : 8;
    const long g = ((long)block * 256 + threadIdx.x) >> SH;
    const int l = threadIdx.x & (L - 1);
    const int n8 = N / 8;
    const bool live = g < (long)M * n8;   // whole groups of L lanes are live or not; all lanes take part in the shuffles
    const long gg = live ? g : 0;
    const int m = (int)(gg / n8), n0 = (int)(gg - (long)m * n8) * 8;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const long stride = (long)M * N;
    const float *p0 = ws + (long)m * N + n0;
    int s = l;
    for (; s + 3 * L < splits; s += 4 * L) {   // four partials in flight
        float4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float4 *p = reinterpret_cast<const float4 *>(p0 + (s + L * u) * stride);
            a[u] = p[0]; b[u] = p[1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[0] += a[u].x; v[1] += a[u].y; v[2] += a[u].z; v[3] += a[u].w;
            v[4] += b[u].x; v[5] += b[u].y; v[6] += b[u].z; v[7] += b[u].w;
        }
    }
    for (; s < splits; s += L) {
        const float4 *p = reinterpret_cast<const float4 *>(p0 + s * stride);
        const float4 a = p[0], b = p[1];
        v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w;
        v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
    }
#pragma unroll
    for (int d = 1; d < L && d < 64; d <<= 1) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] += __shfl_xor(v[r], d, L < 64 ? L : 64);
    }
    if constexpr (L == 256) {
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int r = 0; r < 8; ++r) part[threadIdx.x >> 6][r] = v[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = (part[0][r] + part[1][r]) + (part[2][r] + part[3][r]);
    }
    if (!live || l != 0) return;
    float b8[8];
    load_bias8<T>(ep, n0, b8);
    epilogue8<T>(ep, m, n0, v, b8);
}

// The same for a filter gradient (Epilogue mode 1), whose columns (ky, kx, ci) go to [cout][cin][kh][kw]: a workgroup takes
// all window positions of cb input channels of one output channel, adds the partial sums 16 bytes a lane, exchanges the two
// orders in LDS and writes one contiguous run.  Bound by memory.  The kernel above scatters 4-byte stores (36 bytes apart for
// 3 x 3): 384 -> 384 channels, 7 partials (42 MB) 14.4 us there, 8.5 here; 256 -> 384, 10 partials 10.8 and 8.2; 384 -> 256, 14
// partials 13.8 and 10.7; 5 x 5, 96 -> 256, 17 partials 10.6 and 9.0.
constexpr int kReduceLds = 2048;   // floats: window positions times channels of a workgroup
__device__ __forceinline__ void reduce_filters(const float *ws, int splits, const Epilogue &ep, int M, int N, int npos, int cb_max, int chunks,
                                               unsigned block, float *sums)
{
    const int m = (int)block / chunks, c0 = ((int)block - m * chunks) * cb_max;
    if (m >= ep.cw_cout) return;
    const int cb = min(cb_max, ep.cw_cinp - c0), c4 = cb >> 2;   // channel counts are multiples of 8
    const size_t stride = (size_t)M * N;
    for (int g = threadIdx.x; g < npos * c4; g += blockDim.x) {
        const int pos = g / c4, c = (g - pos * c4) * 4;
        const float *p = ws + (size_t)m * N + pos * ep.cw_cinp + c0 + c;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < splits; s += 8) {   // eight partials in flight; added in split order
            f32x4 a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s + u < splits) a[u] = *reinterpret_cast<const f32x4 *>(p + (size_t)(s + u) * stride);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s + u < splits) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += a[u][e];
                }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) sums[(c + e) * npos + pos] = v[e];
    }
    __syncthreads();
    float *o = static_cast<float *>(ep.out) + ((size_t)m * ep.cw_cin + c0) * npos;
    const int n = min(cb, ep.cw_cin - c0) * npos;
    for (int i = threadIdx.x; i < n; i += blockDim.x) o[i] = sums[i];
}

// LDS of a workgroup
union ReduceShared { float part[4][8]; float sums[kReduceLds]; };
template <typename T> __device__ __forceinline__ void reduce_block(const Reduction &r, unsigned block, ReduceShared &sh)
{
    if (r.lanes == 256) reduce_wide<T, 256>(r.ws, r.splits, r.ep, r.M, r.N, block, sh.part);
    else if (r.lanes == 32) reduce_wide<T, 32>(r.ws, r.splits, r.ep, r.M, r.N, block, sh.part);
    else if (r.lanes == 8) reduce_wide<T, 8>(r.ws, r.splits, r.ep, r.M, r.N, block, sh.part);
    else if (r.lanes == 0) reduce_filters(r.ws, r.splits, r.ep, r.M, r.N, r.npos, r.cb, r.chunks, block, sh.sums);
    else reduce_plain<T>(r.ws, r.splits, r.ep, r.M, r.N, block);
}

}  // namespace asgd
