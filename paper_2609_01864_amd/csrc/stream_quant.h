// stream_quant.h -- the streaming form (stream.h) of the row-wise int8
// quantisation.
//
// The one-row kernel spends 28 instructions an element (4096 x 11008 BF16: 32
// of its 42 us) on rounding, clamping, packing and on proving each code right.
// Here the largest magnitude is an integer maximum of the packed values, and
// the code of x is the low byte of one FMA, x f + 1.5 2^23.
//
// FP32: it is computed for two factors f that enclose 127 / amax; where both give
// the same code it is the exact one, else the vector is decided as before.
//
// BF16: x / amax = m 2^u / m' with whole m, m' < 256, so 127 x / amax is a half (k + 1/2)
// only where x = +-amax / 2 (63.5, to 64) or where m' = 254 (127 / amax is a power of
// two, the product exact); any other lies at least 2^u / 510 from a half, and the
// product's error, 2^-22 of at most 2^(u + 8), never reaches it.  So one factor
// serves: 127 / amax a little enlarged, which turns 63.5 upwards, or itself where
// it is a power of two.  (A tie at amax / 2 is in nearly every second wave's vector
// of normal data, which is what the proof per element cost.)
//
// Rows whose factor is not an ordinary one and lanes that hold a NaN are decided
// as before.
#pragma once
#include "stream.h"

namespace credit {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Largest of the wave's magnitudes: as whole numbers, one instruction a level.
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned dpp_umax(unsigned v) {
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
    return v > o ? v : o;
}
__device__ __forceinline__ float wave_max_mag(float f) {
    unsigned v = __float_as_uint(f);
    v = dpp_umax<0x111, 0xF>(v);
    v = dpp_umax<0x112, 0xF>(v);
    v = dpp_umax<0x114, 0xF>(v);
    v = dpp_umax<0x118, 0xF>(v);
    v = dpp_umax<0x142, 0xA>(v);
    v = dpp_umax<0x143, 0xC>(v);
    return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)v, 63));
}
struct MergeMag {
    __device__ __forceinline__ void operator()(float (&a)[1], const float (&b)[1]) const {
        const unsigned x = __float_as_uint(a[0]), y = __float_as_uint(b[0]);
        a[0] = __uint_as_float(x > y ? x : y);
    }
};

template <> struct StreamStat<OP_QUANT_I8> {
    typedef MergeMag M;
    static constexpr int NS = 1, NX = 1;
    static constexpr float ident = 0.f;  // of magnitudes
};

template <int DT, int V, int R, bool FULL, bool SPLIT>
__device__ __forceinline__ void stream_quant_rows(const RowArgs &a, int c, int grp, StreamLds<OP_QUANT_I8, R> &lds) {
    constexpr int OP = OP_QUANT_I8, EPV = Io<DT>::EPV, B = Io<DT>::BYTES;
    const int tid = threadIdx.x, T = (int)blockDim.x;
    int parity = 0;
    // the slice, as in stream.h
    const int64_t c0 = (int64_t)c * a.chunk;
    const int64_t left = a.N - c0;
    const int nval = (int)(left <= 0 ? 0 : left < a.chunk ? left : a.chunk);
    const int nfv = nval / EPV, tn = nval - nfv * EPV;
    const int jp = nfv / T;
    const uint32_t rowlast = (uint32_t)(a.N * B) - 16u;
    constexpr int VO = FULL ? 1 : V;
    uint32_t off[VO];
#pragma unroll
    for (int j = 0; j < VO; ++j) {
        const uint32_t o = (uint32_t)(c0 * B) + (uint32_t)(j * T + tid) * 16u;
        off[j] = FULL || o < rowlast ? o : rowlast;
    }
    auto step_of = [&](int j) -> uint32_t { return FULL ? (uint32_t)(j * T) * 16u : 0u; };
    auto vo = [](int j) -> int { return FULL ? 0 : j; };
    const int vjp = jp * T + tid;
    const bool lane_full = vjp < nfv, lane_part = vjp == nfv && tn > 0;
    const int lo = lane_part ? EPV - tn : 0;
    const bool wave_full = __builtin_amdgcn_ballot_w64(lane_full) == ~0ull;  // in slot jp

    u32x4 x[R][V], n[R][V];
    auto issue = [&](int64_t row0, uint32_t live) {
        uint32_t o[VO];
#pragma unroll
        for (int j = 0; j < VO; ++j) {
            o[j] = off[j] & live;
            asm volatile("" : "+v"(o[j]));
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t row = row0 + i < a.M ? row0 + i : row0;
            const char *r0 = (const char *)a.in0 + row * a.ld0 * B;
#pragma unroll
            for (int j = 0; j < V; ++j) n[i][j] = vload_nt<false>(r0 + (step_of(j) & live), o[vo(j)]);
        }
    };
    // elements that are not the lane's own count as 0
    auto mask = [&](u32x4 &d, int j) {
        if constexpr (!FULL) {
            if (j < jp || (j == jp && wave_full)) return;
            if (j > jp) {
                d = u32x4{0u, 0u, 0u, 0u};
                return;
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                auto own = [&](int i) -> bool { return (lane_full || lane_part) && i >= lo; };
                if constexpr (B == 4) d[w] = own(w) ? d[w] : 0u;
                else d[w] &= (own(2 * w) ? 0xffffu : 0u) | (own(2 * w + 1) ? 0xffff0000u : 0u);
            }
        }
    };
    uint32_t so[VO];  // off / B, made opaque every round
    // one byte per element; unconditional buffer stores as in stream.h
    auto store = [&](int64_t row, bool live, int j, const unsigned (&w)[EPV / 4]) {
        char *orow = (char *)a.out + row * a.ldo;
        __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            orow + step_of(j) / B, 0, live ? (int)((uint32_t)a.N - step_of(j) / B) : 0, 0x00020000);
        const bool full = FULL || j < jp || (j == jp && lane_full);
        const uint32_t at = full ? so[vo(j)] : 0x80000000u;
        constexpr int AUX = CREDIT_STORE_NT ? 2 : 0;
        if constexpr (EPV == 8) {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, rs, at, 0, AUX);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(w[0], rs, at, 0, AUX);
        }
        if (!FULL && live && j == jp && lane_part) {
#pragma unroll
            for (int i = 1; i < EPV; ++i)
                if (i >= lo) (orow + so[vo(j)])[i] = (char)(w[i / 4] >> (8 * (i & 3)));
        }
    };

    const int64_t step = (int64_t)a.groups * R;
    int64_t row0 = (int64_t)grp * R;
    if (row0 < a.M) issue(row0, 0xffffffffu);
    __builtin_amdgcn_s_waitcnt(0);  // the loop's own waits then count its own accesses only
    for (; row0 < a.M; row0 += step) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < V; ++j) x[i][j] = n[i][j];
        const int64_t nrow = row0 + step;
        issue(nrow < a.M ? nrow : row0, nrow < a.M ? 0xffffffffu : 0u);
        __builtin_amdgcn_sched_barrier(0);
        const int nr = (int)(a.M - row0 < R ? a.M - row0 : R);
#pragma unroll
        for (int j = 0; j < VO; ++j) {
            so[j] = off[j] / B;
            asm volatile("" : "+v"(so[j]));
        }
        float st[R][1];
        bool odd[R];  // the lane holds a NaN
#pragma unroll
        for (int i = 0; i < R; ++i) {
            float am;
            if constexpr (B == 4) {
                unsigned m = 0u;
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    mask(x[i][j], j);
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const unsigned u = x[i][j][w] & 0x7fffffffu;
                        m = m > u ? m : u;
                    }
                }
                am = __uint_as_float(m);
            } else {
                u16x2 m = {0, 0};
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    mask(x[i][j], j);
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, x[i][j][w] & 0x7fff7fffu));
                }
                am = __uint_as_float((unsigned)(m[0] > m[1] ? m[0] : m[1]) << 16);
            }
            odd[i] = am != am;
            if (odd[i]) {  // the largest of the others
                am = 0.f;
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    float q[EPV];
                    decode<DT>(x[i][j], q, 1.f);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) am = fmaxf(am, fabsf(q[e]));
                }
            }
            st[i][0] = wave_max_mag(am);
        }
        stream_reduce<OP, R, SPLIT>(st, a, row0, nr, c, lds, parity);
#pragma unroll
        for (int i = 0; i < R; ++i) opaque<V>(x[i]);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float amx = st[i][0];
            float sc = 1.f, inv = 1.f;  // an all-zero row: every code is 0
            if (amx > 0.f) quant_row_factors(amx, 127.f, sc, inv);
            const bool plain = amx == 0.f || (amx >= 0x1p-100f && amx < INFINITY);
            // 127 / amax lies between these (inv is it, rounded).  BF16 needs the
            // larger only, or inv itself where it is a power of two (above).
            const bool pow2 = (__float_as_uint(inv) & 0x7fffffu) == 0u;
            const float inv_lo = inv * (1.f - 0x1p-22f), inv_hi = B == 2 && pow2 ? inv : inv * (1.f + 0x1p-22f);
            if (c == 0 && tid == 0 && i < nr) a.so[row0 + i] = amx > 0.f ? amx / 127.f : 1.f;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                float q[EPV];
                decode<DT>(x[i][j], q, 1.f);
                unsigned w[EPV / 4];
                unsigned differ = 0u;
#pragma unroll
                for (int e = 0; e < EPV; e += 4) {
                    float t[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        t[u] = fmaf(q[e + u], inv_hi, 0x1.8p23f);
                        if constexpr (B == 4)
                            differ |= __float_as_uint(t[u]) ^ __float_as_uint(fmaf(q[e + u], inv_lo, 0x1.8p23f));
                    }
                    w[e / 4] = __builtin_amdgcn_perm(__float_as_uint(t[1]), __float_as_uint(t[0]), 0x0c0c0400u) |
                               __builtin_amdgcn_perm(__float_as_uint(t[3]), __float_as_uint(t[2]), 0x04000c0cu);
                }
                if (!plain || odd[i] || differ)
                    quant_codes_exact<true, EPV>(q, sc, inv, amx > 0.f ? amx : 1.f, w);
                store(row0 + i, i < nr, j, w);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

// FULL: every slice holds exactly V vectors per thread (N = k V T vectors).
template <int DT, int V, int R, bool SPLIT, bool FULL>
__global__ __launch_bounds__(64 * kStreamWaves) void k_stream_quant(RowArgs a) {
    if (SPLIT && a.epoch == 0u && a.epoch_ptr)
        a.epoch = __hip_atomic_load(a.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __shared__ StreamLds<OP_QUANT_I8, R> lds;
    int c = 0, grp = blockIdx.x;
    if constexpr (SPLIT) member_of(a, blockIdx.x, c, grp);
    stream_quant_rows<DT, V, R, FULL, SPLIT>(a, c, grp, lds);
}

}  // namespace credit
