// codec.hip -- the elementwise codecs: FP32 -> dtype and back, with an
// optional per-row scale (code = RNE(x / scale[row]), value = code * scale[row]).
//
// Both are bound by HBM (5 bytes per element with e4m3 codes).  The matrix is
// packed, so the kernels walk it flat: a workgroup takes 1024 * U consecutive
// elements, a thread U groups of four, 256 groups apart.  Every access is then
// aligned and whole (16 bytes of FP32, 4 / 8 / 16 of codes), whatever the row
// width, and U of them are in flight per thread.  Only the row of a group
// depends on the width: the workgroup's first row comes from one multiplication
// by the host's reciprocal of N, a group's row from a comparison (rows of at
// least a workgroup's elements) or a 32-bit multiplication.  The form before
// (one element per thread, byte-sized code accesses, a 64-bit division per
// element) took 105-113 us to encode and 161-180 us to decode 4096 x 16384
// e4m3; this one takes 62.7 and 57.5 us (5.35 and 5.83 TB/s; the copy kernel
// reaches 6.45).  Encoding spends the rest on its correctly rounded divisions.
#include "device.h"

namespace credit {

constexpr int kCodecU = 4;  // groups of four elements per thread

// Codes of four consecutive elements: 16, 8 or 4 bytes.
template <int DT> struct Code4;
template <> struct Code4<DT_F32> { typedef u32x4 T; };
template <> struct Code4<DT_BF16> { typedef unsigned T __attribute__((ext_vector_type(2))); };
template <> struct Code4<DT_FP8> { typedef unsigned T; };

template <int DT> __device__ __forceinline__ typename Code4<DT>::T encode4(const float *v) {
    typename Code4<DT>::T c;
    if constexpr (DT == DT_F32) {
        c = encode<DT_F32>(v, 1.f);
    } else if constexpr (DT == DT_BF16) {
        c[0] = bf16_bits(v[0]) | (bf16_bits(v[1]) << 16);
        c[1] = bf16_bits(v[2]) | (bf16_bits(v[3]) << 16);
    } else {
        int w = __builtin_amdgcn_cvt_pk_fp8_f32(sat448(v[0]), sat448(v[1]), 0, false);
        c = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(sat448(v[2]), sat448(v[3]), w, true);
    }
    return c;
}
template <int DT> __device__ __forceinline__ void decode4(typename Code4<DT>::T c, float *v) {
    if constexpr (DT == DT_F32) {
        decode<DT_F32>(c, v, 1.f);
    } else if constexpr (DT == DT_BF16) {
        v[0] = __uint_as_float(c[0] << 16);
        v[1] = __uint_as_float(c[0] & 0xffff0000u);
        v[2] = __uint_as_float(c[1] << 16);
        v[3] = __uint_as_float(c[1] & 0xffff0000u);
    } else {
        const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)c, false);
        const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)c, true);
        v[0] = lo.x; v[1] = lo.y; v[2] = hi.x; v[3] = hi.y;
    }
}

// Rows of a packed matrix's elements.  rn64 = floor((2^64 - 1) / N), the row
// of a workgroup's first element is exact after one correction; rn32 =
// ceil(2^32 / N) for N < kCodecSpan, exact for offsets below 2 * kCodecSpan
// (offset * (rn32 * N - 2^32) < 2^32); rn32 = 0 for wider rows, where a
// workgroup meets at most one boundary.
constexpr int kCodecSpan = 256 * 4 * kCodecU;
struct RowWalk {
    int64_t M, N;
    uint64_t rn64;
    uint32_t rn32;
    int64_t row0, r0;  // row of the workgroup's first element, its column
    __device__ __forceinline__ void start(int64_t e0) {
        uint64_t q = __umul64hi((uint64_t)e0, rn64);
        int64_t r = e0 - (int64_t)q * N;
        if (r >= N) { ++q; r -= N; }
        row0 = (int64_t)q;
        r0 = r;
    }
    // scales of the four elements at offset `off` from the first
    __device__ __forceinline__ void scales(const float *scale, int off, float *s) const {
        int64_t row, col;
        if (rn32) {
            const uint32_t o = (uint32_t)r0 + (uint32_t)off, q = __umulhi(o, rn32);
            row = row0 + q;
            col = o - q * (uint32_t)N;
        } else {
            const bool next = r0 + off >= N;
            row = row0 + (next ? 1 : 0);
            col = r0 + off - (next ? N : 0);
        }
        s[0] = scale[row];
        s[1] = s[2] = s[3] = s[0];
        if (col + 3 >= N) {  // the group ends a row; N >= 4: one boundary at most
            const float n = row + 1 < M ? scale[row + 1] : s[0];
#pragma unroll
            for (int i = 1; i < 4; ++i)
                if (col + i >= N) s[i] = n;
        }
    }
};

// N >= 4, both pointers 16-byte aligned (codes: to the size of four).
template <int DT, bool ENC>
__global__ __launch_bounds__(256) void k_codec4(const void *src, const float *scale, void *dst, RowWalk rw) {
    typedef typename Code4<DT>::T CT;
    const int64_t total = rw.M * rw.N, groups = total >> 2;
    const int64_t g0 = (int64_t)blockIdx.x * (256 * kCodecU);
    if (scale) rw.start(g0 * 4);
    u32x4 f[kCodecU];
    CT c[kCodecU];
#pragma unroll
    for (int u = 0; u < kCodecU; ++u) {
        const int64_t g = g0 + u * 256 + threadIdx.x;
        if (g < groups) {
            if constexpr (ENC) f[u] = __builtin_nontemporal_load((const u32x4 *)src + g);
            else c[u] = __builtin_nontemporal_load((const CT *)src + g);
        }
    }
#pragma unroll
    for (int u = 0; u < kCodecU; ++u) {
        const int o = u * 256 + (int)threadIdx.x;
        if (g0 + o >= groups) continue;
        float v[4], s[4];
        if (scale) rw.scales(scale, 4 * o, s);
        if constexpr (ENC) {
            decode<DT_F32>(f[u], v, 1.f);
            if (scale)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = v[i] / s[i];
            __builtin_nontemporal_store(encode4<DT>(v), (CT *)dst + g0 + o);
        } else {
            decode4<DT>(c[u], v);
            if (scale)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = v[i] * s[i];
            __builtin_nontemporal_store(encode<DT_F32>(v, 1.f), (u32x4 *)dst + g0 + o);
        }
    }
}

// One element per thread: the last total % 4 elements of the form above, and
// whole matrices with rows of under four elements or unaligned pointers.
template <int DT>
__global__ __launch_bounds__(256) void k_encode(const float *x, const float *scale, void *out, int64_t M, int64_t N,
                                                int64_t first) {
    const int64_t total = M * N;
    for (int64_t i = first + (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        float v = x[i];
        if (scale) v = v / scale[i / N];
        if constexpr (DT == DT_F32) {
            ((float *)out)[i] = v;
        } else if constexpr (DT == DT_BF16) {
            ((unsigned short *)out)[i] = (unsigned short)bf16_bits(v);
        } else {
            int w = __builtin_amdgcn_cvt_pk_fp8_f32(sat448(v), 0.f, 0, false);
            ((unsigned char *)out)[i] = (unsigned char)(w & 0xff);
        }
    }
}
template <int DT>
__global__ __launch_bounds__(256) void k_decode(const void *in, const float *scale, float *out, int64_t M, int64_t N,
                                                int64_t first) {
    const int64_t total = M * N;
    for (int64_t i = first + (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        float v;
        if constexpr (DT == DT_F32) {
            v = ((const float *)in)[i];
        } else if constexpr (DT == DT_BF16) {
            v = __uint_as_float((unsigned)((const unsigned short *)in)[i] << 16);
        } else {
            f32x2 t = __builtin_amdgcn_cvt_pk_f32_fp8((int)((const unsigned char *)in)[i], false);
            v = t.x;
        }
        out[i] = scale ? v * scale[i / N] : v;
    }
}

template <int DT, bool ENC>
static hipError_t codec(int64_t M, int64_t N, const void *src, const float *scale, void *dst, hipStream_t s) {
    const int64_t total = M * N;
    const uintptr_t code = (uintptr_t)(ENC ? dst : src), real = (uintptr_t)(ENC ? (uintptr_t)src : (uintptr_t)dst);
    const int64_t blocks = (total / 4 + 256 * kCodecU - 1) / (256 * kCodecU);
    int64_t first = 0;  // elements the grouped form covers
    if (N >= 4 && real % 16 == 0 && code % sizeof(typename Code4<DT>::T) == 0 && blocks > 0 && blocks < (1LL << 31)) {
        RowWalk rw{};
        rw.M = M;
        rw.N = N;
        rw.rn64 = ~0ull / (uint64_t)N;
        rw.rn32 = N < kCodecSpan ? (uint32_t)(((1ull << 32) + N - 1) / N) : 0u;
        void *args[] = {&src, &scale, &dst, &rw};
        const hipError_t e =
            hipLaunchKernel((const void *)&k_codec4<DT, ENC>, dim3((unsigned)blocks), dim3(256), args, 0, s);
        first = total / 4 * 4;
        if (e != hipSuccess || first == total) return e;
    }
    int64_t grid = (total - first + 255) / 256;
    if (grid > 8192) grid = 8192;
    const void *fn = nullptr;
    if constexpr (ENC) fn = (const void *)&k_encode<DT>;
    else fn = (const void *)&k_decode<DT>;
    void *args[] = {&src, &scale, &dst, &M, &N, &first};
    return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(256), args, 0, s);
}

// Launches the codec of a packed [M, N] matrix (M, N > 0) on stream s.
hipError_t launch_encode(int dt, int64_t M, int64_t N, const float *x, const float *scale, void *out, hipStream_t s) {
    return dt == DT_F32 ? codec<DT_F32, true>(M, N, x, scale, out, s)
         : dt == DT_BF16 ? codec<DT_BF16, true>(M, N, x, scale, out, s) : codec<DT_FP8, true>(M, N, x, scale, out, s);
}
hipError_t launch_decode(int dt, int64_t M, int64_t N, const void *in, const float *scale, float *out, hipStream_t s) {
    return dt == DT_F32 ? codec<DT_F32, false>(M, N, in, scale, out, s)
         : dt == DT_BF16 ? codec<DT_BF16, false>(M, N, in, scale, out, s) : codec<DT_FP8, false>(M, N, in, scale, out, s);
}

}  // namespace credit
