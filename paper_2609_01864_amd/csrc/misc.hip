// misc.hip -- support kernels: dgamma/dbeta column reductions, the work-free
// control kernel of the profitability model, cache flush, deterministic fill
// and the copy-bandwidth probe.
#include "resident.h"
#include "twopass.h"

namespace credit {

// out_p[j] = sum over g < parts of part[g][p][j]: a workgroup takes CW columns
// of one p, its S slices of CW threads each add every S-th partial row (eight
// loads in flight), and the slices are added in order through LDS
// (deterministic: no atomics, fixed order).  One launch with rows of the
// partials spread over S threads: as two launches of one column per thread
// (slices of 16 rows, then the slices) the second ran N / 256 workgroups, each
// a serial chain, and the pair took 40 us for 768 partial rows of 2 x 4096
// columns; this takes 5.4 us.  32 columns (a 128-byte line of each row) by 32
// slices while that leaves the chip idle, else 64 by 4.
template <int CW, int S>
__global__ __launch_bounds__(CW * S) void k_colreduce(const float *part, int parts, int ncp, int64_t N, float *out0,
                                                      float *out1) {
    __shared__ float sums[S][CW];
    float *o = blockIdx.y == 0 ? out0 : out1;
    if (!o) return;
    const int col = threadIdx.x % CW, sl = threadIdx.x / CW;
    const int64_t j = (int64_t)blockIdx.x * CW + col;
    float s = 0.f;
    if (j < N) {
        const float *p = part + (int64_t)blockIdx.y * N + j;
        const int64_t ld = (int64_t)ncp * N;
        int g = sl;
        for (; g + 7 * S < parts; g += 8 * S) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[(g + u * S) * ld];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; g < parts; g += S) s += p[g * ld];
    }
    sums[sl][col] = s;
    __syncthreads();
    if (sl == 0 && j < N) {
#pragma unroll
        for (int u = 1; u < S; ++u) s += sums[u][col];
        o[j] = s;
    }
}

hipError_t launch_colreduce(const float *part, int parts, int ncp, int64_t N, float *out0, float *out1, hipStream_t st) {
    const bool narrow = N * ncp < 32 * 2048;
    const int cw = narrow ? 32 : 64;
    void *args[] = {&part, &parts, &ncp, &N, &out0, &out1};
    return hipLaunchKernel(narrow ? (const void *)&k_colreduce<32, 32> : (const void *)&k_colreduce<64, 4>,
                           dim3((unsigned)((N + cw - 1) / cw), ncp), dim3(narrow ? 1024 : 256), args, 0, st);
}

const void *colstats_kernel(int dt, bool ln) {
    if (dt == DT_F32) return ln ? (const void *)&k_colstats<DT_F32, true> : (const void *)&k_colstats<DT_F32, false>;
    if (dt == DT_BF16) return ln ? (const void *)&k_colstats<DT_BF16, true> : (const void *)&k_colstats<DT_BF16, false>;
    if (dt == DT_FP8) return ln ? (const void *)&k_colstats<DT_FP8, true> : (const void *)&k_colstats<DT_FP8, false>;
    return nullptr;
}

// The work-free control kernel (Sec. III-D): the split-row kernel's grid, row
// groups, split factor and occupancy (pinned through the dynamic LDS size
// chosen by the host), and per row `stages` workgroup barriers plus, for
// k > 1, the partial exchange; no row data is read or written.
__global__ __launch_bounds__(kBlock) void k_control(RowArgs a, int stages) {
    extern __shared__ float pin[];
    __shared__ float red[2 * 4 * 2];
    __shared__ float xb[kMaxK * kMaxQ];
    int parity = 0;
    int c, grp;
    member_of(a, blockIdx.x, c, grp);
    for (int64_t row = grp; row < a.M; row += a.groups) {
        for (int s = 0; s < stages; ++s) {
            float v[2] = {(float)threadIdx.x, 0.f};
            block_reduce<4, 2>(v, MergeSum(), red, parity);
            if (a.k > 1) exchange<2>(a, row, s, c, v, xb);
        }
    }
    if (a.M < 0) pin[threadIdx.x] = red[0];  // keeps the dynamic allocation
}

const void *control_kernel() { return (const void *)&k_control; }

// Zero-fill of n 32-bit words (used instead of a memset node so the sequence
// stays safe under stream capture).
__global__ __launch_bounds__(256) void k_zero(unsigned *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0u;
}
const void *zero_kernel() { return (const void *)&k_zero; }

// Advances the device-side exchange epoch of graph-recorded launches.  These
// epochs have the top bit set and host-chosen epochs have it clear, so the two
// never coincide; the 31-bit count wraps and never yields 0.
__global__ void k_epoch_bump(unsigned *ctr) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const unsigned e = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned n = ((e + 1u) & 0x7fffffffu) | 0x80000000u;
        __hip_atomic_store(ctr, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
const void *epoch_bump_kernel() { return (const void *)&k_epoch_bump; }

// Cache flush by reading: streams n 16-byte vectors so the L2s and the
// Infinity Cache hold clean lines of this buffer, not the operator's data
// (a write sweep would leave dirty lines to be written back during the
// timed kernel).  The sink is written only on an impossible sum.
__global__ __launch_bounds__(256) void k_flush_read(const u32x4 *__restrict__ p, int64_t n, unsigned *sink) {
    unsigned acc = 0u;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        u32x4 v = p[i];
        acc ^= v[0] ^ v[1] ^ v[2] ^ v[3];
    }
    if (acc == 0x9e3779b9u && threadIdx.x == 0x1ff) sink[0] = acc;
}
const void *flush_kernel() { return (const void *)&k_flush_read; }

// Deterministic pseudo-random fill of a timing buffer with values valid for
// the dtype: FP32 / BF16 in [-2, 2), FP8 any finite code.
__device__ __forceinline__ unsigned mix32(unsigned long long x) {
    x ^= x >> 33;
    x *= 0xff51afd7ed558ccdULL;
    x ^= x >> 33;
    x *= 0xc4ceb9fe1a85ec53ULL;
    x ^= x >> 33;
    return (unsigned)x;
}
__global__ __launch_bounds__(256) void k_fill(unsigned *p, int64_t nwords, unsigned seed, int dt) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nwords; i += (int64_t)gridDim.x * 256) {
        unsigned h = mix32(((unsigned long long)seed << 40) ^ (unsigned long long)i);
        unsigned w;
        if (dt == DT_F32) {
            w = __float_as_uint(((float)(h >> 8) * (1.f / 16777216.f)) * 4.f - 2.f);
        } else if (dt == DT_BF16) {
            float a = ((float)(h & 0xffff) * (1.f / 65536.f)) * 4.f - 2.f;
            float b = ((float)(h >> 16) * (1.f / 65536.f)) * 4.f - 2.f;
            w = (__float_as_uint(a) >> 16) | (__float_as_uint(b) & 0xffff0000u);
        } else {
            w = h;
            // replace NaN codes (S.1111.111) by the largest finite code
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (((w >> (8 * b)) & 0x7fu) == 0x7fu) w ^= 1u << (8 * b);
        }
        p[i] = w;
    }
}
const void *fill_kernel() { return (const void *)&k_fill; }

// Streaming copy used to calibrate the achievable read+write bandwidth and the
// hardware traffic counters.
__global__ __launch_bounds__(256) void k_copy(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int64_t n) {
    // one 16-byte vector per work-item over a grid that covers the buffer:
    // the hardware dispatcher streams workgroups through the CUs, which
    // measured faster than any grid-stride or multi-vector form
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}
const void *copy_kernel() { return (const void *)&k_copy; }

}  // namespace credit
