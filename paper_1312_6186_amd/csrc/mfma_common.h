// Device-side pieces shared by the kernels that multiply on the matrix cores: element
// types, range-checked 16-byte operand loads, fragments, and what happens to an
// accumulator on its way to memory.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "asgd_internal.h"

namespace asgd {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16_t;

template <typename T> struct Geo;
template <> struct Geo<bf16_t> { enum { CH = 8, BK = 64, KSTEPS = 4 }; };
template <> struct Geo<float> { enum { CH = 4, BK = 32, KSTEPS = 2 }; };

#define ASGD_INLINE __attribute__((always_inline))

// Compile-time loop: indices reach the body as constants, so register arrays are never addressed dynamically.
template <int I, int N, class F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv &f) { return (__umulhi(n, f.mul) + n) >> f.sh; }
__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }

// All operand fetches are 16-byte buffer loads: the operand tensor is described to the hardware as a byte range,
// a lane passes a 32-bit byte offset, and an offset outside the range returns zeros.  A loader therefore never
// builds a 64-bit address and never branches: pieces that must read as zero (rows or K positions past the end,
// window positions outside the image) get an offset with the top two bits set.  Offsets of valid pieces stay
// below 1 GiB (checked on the host), so the sum of a valid and an invalid part is still out of range.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kInv = 0xC0000000u;
constexpr unsigned kMaxOperandBytes = 0x40000000u;

struct Operand {
    const void *base; unsigned bytes;
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc() const
    {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
    }
};
template <bool NONTEMPORAL = false> __device__ __forceinline__ uint4 buf_ld16(__amdgpu_buffer_rsrc_t rs, unsigned off)
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, NONTEMPORAL ? 2 : 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}
// LDS tile of a row-contiguous operand: BK lines of ROWS elements.  A transposing read makes half a wave touch
// 4 K lines x 64 bytes; with lines 64 bytes (mod 256) apart those eight 32-byte groups cover all banks once.
template <typename T, int ROWS> struct TransTile {
    static constexpr int LINE = ROWS * (int)sizeof(T) + (sizeof(T) == 4 ? 32 : ROWS == 32 ? 128 : 64);   // bytes
    static constexpr int BYTES = Geo<T>::BK * LINE;
};

// ------------------------------------------------------------------ MFMA step
// A fragment is the 8 consecutive K elements of one row that a lane feeds to the
// MFMA.  FragOff holds, per K step, the LDS byte offset of that piece for the
// lane's row in row block 0 and in row block 1 (blocks 64 rows apart share it), so
// the inner loop issues its LDS reads with no address arithmetic.
template <typename T> struct Frag;
template <typename T, bool TRANS, int ROWS> struct FragOff;
template <int ROWS> struct FragOff<bf16_t, false, ROWS> {
    unsigned o[Geo<bf16_t>::KSTEPS][2];
    __device__ __forceinline__ void init(int row0, int lane)
    {
        const int lrow = lane & 31, half = lane >> 5;
        static_for<0, Geo<bf16_t>::KSTEPS>([&](auto ks) ASGD_INLINE {
            static_for<0, 2>([&](auto par) ASGD_INLINE {
                const int row = row0 + par * 32 + lrow;
                o[ks][par] = (unsigned)(row * 8 + ((ks * 2 + half) ^ swz(row))) * 16u;
            });
        });
    }
};
template <int ROWS> struct FragOff<float, false, ROWS> {
    unsigned o[Geo<float>::KSTEPS][2][2];
    __device__ __forceinline__ void init(int row0, int lane)
    {
        const int lrow = lane & 31, half = lane >> 5;
        static_for<0, Geo<float>::KSTEPS>([&](auto ks) ASGD_INLINE {
            static_for<0, 2>([&](auto par) ASGD_INLINE {
                const int row = row0 + par * 32 + lrow, q = ks * 4 + half * 2, z = swz(row);
                o[ks][par][0] = (unsigned)(row * 8 + (q ^ z)) * 16u;
                o[ks][par][1] = (unsigned)(row * 8 + ((q + 1) ^ z)) * 16u;
            });
        });
    }
};
// Row-contiguous tiles.  16-bit data: ds_read_b64_tr_b16 works on blocks of 16 lanes; when lane j of a block
// points at K line (j >> 2) and row piece (j & 3) of a 4 x 16 patch, lane i receives row i of the patch for the
// four K lines in order.  Lane L = 16*b + i of the wave wants row 16*(b & 1) + i and K lines 8*(b >> 1) + 0..7
// of the K step, i.e. two such reads.  32-bit data needs no hardware help: eight 4-byte reads down the K axis.
template <int ROWS> struct FragOff<bf16_t, true, ROWS> {
    unsigned base;
    __device__ __forceinline__ void init(int row0, int lane)
    {
        const int b = lane >> 4, i = lane & 15;
        base = (unsigned)((8 * (b >> 1) + (i >> 2)) * TransTile<bf16_t, ROWS>::LINE + (row0 + 16 * (b & 1) + 4 * (i & 3)) * 2);
    }
};
template <int ROWS> struct FragOff<float, true, ROWS> {
    unsigned base;
    __device__ __forceinline__ void init(int row0, int lane)
    {
        base = (unsigned)(8 * (lane >> 5) * TransTile<float, ROWS>::LINE + (row0 + (lane & 31)) * 4);
    }
};
typedef short short4v __attribute__((ext_vector_type(4)));
template <> struct Frag<bf16_t> {
    uint4 v;
    template <int KS, int BLK, int ROWS> __device__ __forceinline__ void read(const char *sm, const FragOff<bf16_t, false, ROWS> &fo)
    {
        v = *reinterpret_cast<const uint4 *>(sm + fo.o[KS][BLK % 2] + (BLK / 2) * (64 * 128));
    }
    template <int KS, int BLK, int ROWS> __device__ __forceinline__ void read(const char *sm, const FragOff<bf16_t, true, ROWS> &fo)
    {
        constexpr int LINE = TransTile<bf16_t, ROWS>::LINE;
        typedef __attribute__((address_space(3))) short4v lds_s4;
        const char *p = sm + fo.base + KS * 16 * LINE + BLK * 64;
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(p));
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(p + 4 * LINE));
        const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
        v = make_uint4(a.x, a.y, b.x, b.y);
    }
};
template <> struct Frag<float> {
    uint4 v[2];
    template <int KS, int BLK, int ROWS> __device__ __forceinline__ void read(const char *sm, const FragOff<float, false, ROWS> &fo)
    {
        v[0] = *reinterpret_cast<const uint4 *>(sm + fo.o[KS][BLK % 2][0] + (BLK / 2) * (64 * 128));
        v[1] = *reinterpret_cast<const uint4 *>(sm + fo.o[KS][BLK % 2][1] + (BLK / 2) * (64 * 128));
    }
    template <int KS, int BLK, int ROWS> __device__ __forceinline__ void read(const char *sm, const FragOff<float, true, ROWS> &fo)
    {
        constexpr int LINE = TransTile<float, ROWS>::LINE;
        const char *p = sm + fo.base + KS * 16 * LINE + BLK * 128;
        uint32_t e[8];
        static_for<0, 8>([&](auto j) ASGD_INLINE { e[j] = *reinterpret_cast<const uint32_t *>(p + j * LINE); });
        v[0] = make_uint4(e[0], e[1], e[2], e[3]);
        v[1] = make_uint4(e[4], e[5], e[6], e[7]);
    }
};

__device__ __forceinline__ void mma(f32x16 &acc, const Frag<bf16_t> &first, const Frag<bf16_t> &second)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, first.v), __builtin_bit_cast(bf16x8, second.v),
                                                  acc, 0, 0, 0);
}
__device__ __forceinline__ void mma(f32x16 &acc, const Frag<float> &first, const Frag<float> &second)
{
    const uint32_t a[8] = {first.v[0].x, first.v[0].y, first.v[0].z, first.v[0].w, first.v[1].x, first.v[1].y, first.v[1].z, first.v[1].w};
    const uint32_t b[8] = {second.v[0].x, second.v[0].y, second.v[0].z, second.v[0].w, second.v[1].x, second.v[1].y, second.v[1].z, second.v[1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e]), __uint_as_float(b[e]), acc, 0, 0, 0);
}

// ------------------------------------------------------------------ epilogue
__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

// Store of 8 consecutive output elements (32 bytes fp32 / 16 bytes bf16) as 16-byte vectors: every output
// row starts 16-byte aligned and has a multiple of 8 elements (checked on the host).
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename T> __device__ __forceinline__ void store8(T *p, const float (&v)[8]);
template <> __device__ __forceinline__ void store8<float>(float *p, const float (&v)[8])
{
    f32x4 *q = reinterpret_cast<f32x4 *>(__builtin_assume_aligned(p, 16));
    q[0] = f32x4{v[0], v[1], v[2], v[3]};
    q[1] = f32x4{v[4], v[5], v[6], v[7]};
}
template <> __device__ __forceinline__ void store8<bf16_t>(bf16_t *p, const float (&v)[8])
{
    union { bf16_t h[8]; u32x4 u; } t;
#pragma unroll
    for (int r = 0; r < 8; ++r) t.h[r] = (bf16_t)v[r];
    *reinterpret_cast<u32x4 *>(__builtin_assume_aligned(p, 16)) = t.u;
}

template <typename T> struct Vec8;
template <> struct Vec8<float> { union { float4 u[2]; float e[8]; }; };
template <> struct Vec8<bf16_t> { union { uint4 u[1]; bf16_t e[8]; }; };

// Eight consecutive columns n0..n0+7 of row m (n0 a multiple of 8, all in range).
// The bias of these 8 columns, as fp32 (zeros past bias_n or without a bias).
template <typename T> __device__ __forceinline__ void load_bias8(const Epilogue &ep, int n0, float (&b8)[8])
{
#pragma unroll
    for (int r = 0; r < 8; ++r) b8[r] = 0.f;
    if (ep.bias) {
        const T *b = static_cast<const T *>(ep.bias);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (n0 + r < ep.bias_n) b8[r] = to_f32(b[n0 + r]);
    }
}

template <typename T> __device__ __forceinline__ void epilogue8(const Epilogue &ep, int m, int n0, float (&v)[8], const float (&b8)[8])
{
    if (ep.mode == 1) {  // conv filter gradient: (cout, (ky,kx,ci_padded)) -> canonical [cout][cin][kh][kw]
        if (m >= ep.cw_cout) return;
        const int t = n0 / ep.cw_cinp, ci0 = n0 - t * ep.cw_cinp;
        const int ky = t / ep.cw_kw, kx = t - ky * ep.cw_kw;
        float *o = static_cast<float *>(ep.out);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (ci0 + r < ep.cw_cin) o[(((long)m * ep.cw_cin + ci0 + r) * ep.cw_kh + ky) * ep.cw_kw + kx] = v[r];
        return;
    }
    if (ep.mode == 2) {  // the same for window rows: columns are (ky, j), j = kx*cw_rwc + ci over a padded row of cw_cinp elements
        if (m >= ep.cw_cout) return;
        const int ky = n0 / ep.cw_cinp, j0 = n0 - ky * ep.cw_cinp;
        float *o = static_cast<float *>(ep.out);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int kx = (j0 + r) / ep.cw_rwc, ci = (j0 + r) - kx * ep.cw_rwc;
            if (ci < ep.cw_cin && kx < ep.cw_kw) o[(((long)m * ep.cw_cin + ci) * ep.cw_kh + ky) * ep.cw_kw + kx] = v[r];
        }
        return;
    }
    if (ep.bias) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] += b8[r];
    }
    if (ep.relu) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = v[r] > 0.f ? v[r] : 0.f;
    }
    if (ep.drop) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const uint64_t idx = (uint64_t)m * (uint64_t)ep.drop_F + (uint64_t)(n0 + r);
            const uint32_t u = (uint32_t)(mix64(ep.drop_key + 0x9E3779B97F4A7C15ull * (idx + 1)) >> 32);
            v[r] = (u >= ep.drop_thr) ? v[r] * ep.drop_scale : 0.f;
        }
    }
    if (ep.mask_src) {
        Vec8<T> ms;   // the mask tensor is a workspace tensor: rows and column groups are 16-byte aligned
        const T *mp = static_cast<const T *>(ep.mask_src) + (long)m * ep.mask_ld + n0;
        static_for<0, sizeof(ms.u) / 16>([&](auto i) ASGD_INLINE { ms.u[i] = reinterpret_cast<const std::remove_reference_t<decltype(ms.u[0])> *>(mp)[i]; });
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = to_f32(ms.e[r]) > 0.f ? v[r] * ep.mask_scale : 0.f;
    }
    if (ep.out_f32) {
        // fp32 output = a parameter gradient: read again only by the update, long after it has left every cache
        f32x4 *q = reinterpret_cast<f32x4 *>(__builtin_assume_aligned(static_cast<float *>(ep.out) + (long)m * ep.ld + n0, 16));
        __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, q);
        __builtin_nontemporal_store(f32x4{v[4], v[5], v[6], v[7]}, q + 1);
    }
    else store8<T>(static_cast<T *>(ep.out) + (long)m * ep.ld + n0, v);
}

}  // namespace asgd
