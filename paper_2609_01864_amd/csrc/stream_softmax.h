// stream_softmax.h -- the streaming form (stream.h) of the softmax forward and
// of its backward from the logits.
//
// Nothing is kept from row to row here, so a row's vectors need not start at
// its first element: vector v of a row covers the 16 bytes that begin 16 v - h
// bytes after the row's start, with h = the row's address mod 128 where the
// rows of all its tensors agree on it (contiguous tensors do), else 0.  Every
// access but those at the row's two ends is then aligned, every wave's access
// covers whole 128-byte lines and so does every member's slice, whatever the
// width: the copy of a buffer that is 2 bytes off a line runs at 5.3 TB/s on
// MI355X, an aligned one at 6.3.  The vectors at the ends are loaded as the
// row's first or last 16 bytes with the other elements masked, as in stream.h.
#pragma once
#include "stream.h"

namespace credit {
template <int OP, int DT, int V, int R, bool FULL, bool SPLIT>
__device__ __forceinline__ void stream_softmax_rows(const RowArgs &a, int c, int grp, StreamLds<OP, R> &lds) {
    constexpr int EPV = Io<DT>::EPV, B = Io<DT>::BYTES;
    constexpr bool TWO = two_in(OP), FP8 = DT == DT_FP8;
    typedef StreamStat<OP> S;
    const int tid = threadIdx.x, T = (int)blockDim.x;
    int parity = 0;
    const int nb = (int)(a.N * B), rowlast = nb - 16;
    const int cv = (int)(a.chunk / EPV);         // vectors of a member
    const int v0 = c * cv;                       // its first one
    const int lane0 = (v0 + tid) * 16;           // this thread's byte of slot 0, before the phase
    const int inside = SPLIT ? cv - tid : 0x7fffffff;  // slot j is the member's while j T < inside
    // bytes by which the vectors of a row begin before it
    auto phase = [&](int64_t row) -> int {
        if constexpr (FULL || !stream_phase(OP, V)) return 0;
        const uintptr_t p = (uintptr_t)a.in0 + row * a.ld0 * B, q = (uintptr_t)a.out + row * a.ldo * B;
        bool same = ((p ^ q) & 127u) == 0;
        if constexpr (TWO) same = same && ((p ^ ((uintptr_t)a.in1 + row * a.ld1 * B)) & 127u) == 0;
        return same ? (int)(p & 127u) : 0;
    };
    // offset of slot j in a row of phase h, before it is held inside the row
    auto at = [&](int j, int h) -> int { return lane0 + (j * T * 16 - h); };
    auto held = [&](int o) -> int { return o < 0 ? 0 : o < rowlast ? o : rowlast; };
    auto whole = [&](int j, int h) -> bool {
        const int o = at(j, h);
        return o >= 0 && o <= rowlast && (!SPLIT || j * T < inside);
    };
    // no lane of the workgroup has an element of the slot
    auto empty = [&](int j, int h) -> bool {
        return !FULL && ((SPLIT && j * T >= cv) || (v0 + j * T) * 16 - h >= nb);
    };

    u32x4 x0[R][V], x1[TWO ? R : 1][TWO ? V : 1];
    u32x4 n0[R][V], n1[TWO ? R : 1][TWO ? V : 1];
    float xs[R], nxs[R];  // input scales (FP8)
    // Loads of the round at row0; `live` as in stream.h.
    auto issue = [&](int64_t row0, uint32_t live) {
        uint32_t lb = (uint32_t)lane0 & live;
        asm volatile("" : "+v"(lb));
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t row = row0 + i < a.M ? row0 + i : row0;
            const char *r0 = (const char *)a.in0 + row * a.ld0 * B;
            const char *r1 = TWO ? (const char *)a.in1 + row * a.ld1 * B : nullptr;
            if constexpr (FP8) nxs[i] = a.s0[row];
            if constexpr (FULL) {
#pragma unroll
                for (int j = 0; j < V; ++j) n0[i][j] = vload_nt<false>(r0 + ((uint32_t)(j * T) * 16u & live), lb);
                if constexpr (TWO) {
#pragma unroll
                    for (int j = 0; j < V; ++j) n1[i][j] = vload_nt<false>(r1 + ((uint32_t)(j * T) * 16u & live), lb);
                }
            } else {
                const int h = phase(row);
                uint32_t o[V];
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    o[j] = (uint32_t)held((int)lb + (j * T * 16 - h)) & live;
                    asm volatile("" : "+v"(o[j]));
                }
#pragma unroll
                for (int j = 0; j < V; ++j) n0[i][j] = vload_nt<false>(r0, o[j]);
                if constexpr (TWO) {
#pragma unroll
                    for (int j = 0; j < V; ++j) n1[i][j] = vload_nt<false>(r1, o[j]);
                }
            }
        }
    };
    // which elements of a slot are the lane's own (bytes [lo, hi) of the vector)
    auto bounds = [&](int j, int h, int &lo, int &hi) {
        const int o = at(j, h);
        lo = o > rowlast ? o - rowlast : 0;
        hi = SPLIT && j * T >= inside ? 0 : o < 0 ? o + 16 : 16;
    };
    // `fill` into the elements that are not
    auto mask = [&](u32x4 &d, int j, int h, unsigned fill) {
        if constexpr (!FULL) {
            if (__builtin_amdgcn_ballot_w64(whole(j, h)) == ~0ull) return;
            int lo, hi;
            bounds(j, h, lo, hi);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                unsigned m;
                if constexpr (B == 4) m = 4 * w >= lo && 4 * w < hi ? 0xffffffffu : 0u;
                else
                    m = (4 * w >= lo && 4 * w < hi ? 0xffffu : 0u) |
                        (4 * w + 2 >= lo && 4 * w + 2 < hi ? 0xffff0000u : 0u);
                d[w] = (d[w] & m) | (fill & ~m);
            }
        }
    };
    // Unconditional buffer stores, dropped for lanes without a whole vector
    // (stream.h); the vectors at the row's ends are stored by elements.
    uint32_t sb;  // lane0, made opaque every round
    auto store = [&](int64_t row, bool live, int j, int h, u32x4 v) {
        char *orow = (char *)a.out + row * a.ldo * B;
        if constexpr (FULL) {
            const uint32_t step = (uint32_t)(j * T) * 16u;
            __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(orow + step, 0, live ? (int)((uint32_t)nb - step) : 0, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, sb, 0, CREDIT_STORE_NT ? 2 : 0);
        } else {
            __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(orow, 0, live ? nb : 0, 0x00020000);
            const int o = (int)sb + (j * T * 16 - h);
            const bool ok = o >= 0 && o <= rowlast && (!SPLIT || j * T < inside);
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, ok ? (uint32_t)o : 0x80000000u, 0, CREDIT_STORE_NT ? 2 : 0);
            if (__builtin_amdgcn_ballot_w64(ok) != ~0ull && live && !ok) {
                int lo, hi;
                bounds(j, h, lo, hi);
                char *p = orow + held(o);
#pragma unroll
                for (int i = 0; i < EPV; ++i) {
                    if (i * B < lo || i * B >= hi) continue;
                    if constexpr (B == 4) *(unsigned *)(p + i * B) = v[i];
                    else if constexpr (B == 1) p[i] = (char)(v[i / 4] >> (8 * (i & 3)));
                    else *(unsigned short *)(p + i * B) = (unsigned short)(v[i / 2] >> (16 * (i & 1)));
                }
            }
        }
    };

    const int64_t step = (int64_t)a.groups * R;
    int64_t row0 = (int64_t)grp * R;
    if (row0 < a.M) issue(row0, 0xffffffffu);
    __builtin_amdgcn_s_waitcnt(0);  // the loop's own waits then count its own accesses only
    for (; row0 < a.M; row0 += step) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
#pragma unroll
            for (int j = 0; j < V; ++j) {
                x0[i][j] = n0[i][j];
                if constexpr (TWO) x1[i][j] = n1[i][j];
            }
            xs[i] = FP8 ? nxs[i] : 1.f;
        }
        const int64_t nrow = row0 + step;
        issue(nrow < a.M ? nrow : row0, nrow < a.M ? 0xffffffffu : 0u);
        __builtin_amdgcn_sched_barrier(0);
        const int nr = (int)(a.M - row0 < R ? a.M - row0 : R);
        int ph[R];
#pragma unroll
        for (int i = 0; i < R; ++i) ph[i] = phase(i < nr ? row0 + i : row0);
        sb = (uint32_t)lane0;
        asm volatile("" : "+v"(sb));
        // each pass decodes the packed rows again (resident.h)
        auto fresh = [&]() {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                opaque<V>(x0[i]);
                if constexpr (TWO) opaque<V>(x1[i]);
            }
        };
        // Exponentials about the wave's maximum c in base-2 units, rounded up to
        // a whole number: 32 - c and the factors 2^(c - c') by which the sums of
        // the waves (and members) are rescaled when merged are then exact (FP8
        // takes it as it is: its largest code, 448, stands for 2^0).  Elements
        // that are not the lane's own are -inf (and their dy 0), so they add nothing.
        //
        // KEEP: the exponentials stay in registers for the output (the exponential
        // is the dearest instruction here: 2048 x 50257 BF16 k = 4 98 -> 91 us, FP8 4096
        // x 65536 113 -> 95, FP32 outputs keep their last bits); short BF16 rows run faster with more
        // workgroups (16384 x 1000: 14.9 against 15.7) and the widest slices have no
        // registers for them.  Kept BF16 exponentials, and FP32 ones of the
        // backward, are 2^(v + 32), so that results down to 2^-158 of the largest
        // keep their value (device.h).
        //
        // A far wave (device.h) first takes its maximum off its elements, where they
        // are: a difference is 0 or so large that any rounding of it will do.
        constexpr bool BW = OP == OP_SMXL_BWD, KEEP = V == 4 || (DT == DT_F32 && !BW);
        constexpr float SH = KEEP && (DT == DT_BF16 || BW) ? kExpShift : 0.f;
        constexpr float USH = SH == 0.f ? 1.f : kExpUnshift;
        constexpr unsigned NINF = DT == DT_F32 ? 0xff800000u : 0xff80ff80u;
        float st[R][S::NS], ct[R];
        float ev[KEEP ? R : 1][KEEP ? V * EPV : 1];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float K = xs[i] * kLog2e;
            float qmax = -INFINITY;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if (empty(j, ph[i])) continue;
                float q[EPV];
                if constexpr (FP8) {
                    // (e4m3 has no infinity to mask with)
                    decode<DT>(x0[i][j], q, 1.f);
                    if (!FULL && __builtin_amdgcn_ballot_w64(whole(j, ph[i])) != ~0ull) {
                        int lo, hi;
                        bounds(j, ph[i], lo, hi);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) q[e] = e >= lo && e < hi ? q[e] : -INFINITY;
                    }
                } else {
                    mask(x0[i][j], j, ph[i], NINF);
                    if constexpr (BW) mask(x1[i][j], j, ph[i], 0u);
                    decode<DT>(x0[i][j], q, 1.f);
                }
#pragma unroll
                for (int e = 0; e < EPV; ++e) qmax = fmaxf(qmax, q[e]);
                keep_order(qmax);
            }
            opaque<V>(x0[i]);
            qmax = wave_max(qmax);
            st[i][0] = FP8 ? base2_ref(qmax, K) : ceilf(base2_ref(qmax, kLog2e));
            const float c0 = qmax == -INFINITY ? 0.f : st[i][0];
            ct[i] = KEEP ? c0 : lane_value(c0, 0);  // (a scalar register, where they are short)
            float cs = SH - ct[i];
            if (!FP8 && __builtin_expect(far_ref(ct[i]), 0)) {
                cs = SH;
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    float q[EPV];
                    asm volatile("" : "+v"(x0[i][j]));  // one at a time: no registers for more
                    decode<DT>(x0[i][j], q, 1.f);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) q[e] -= qmax;
                    x0[i][j] = encode<DT>(q, 1.f);
                    asm volatile("" : "+v"(x0[i][j]));
                }
            }
            float s = 0.f, t = 0.f;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if (empty(j, ph[i])) continue;
                float q[EPV], g[EPV];
                decode<DT>(x0[i][j], q, 1.f);
                if constexpr (BW) decode<DT>(x1[i][j], g, 1.f);
                float x[EPV];
#pragma unroll
                for (int e = 0; e < EPV; ++e) x[e] = fast_exp2(fmaf(q[e], FP8 ? K : kLog2e, cs));
                if constexpr (FP8 && !FULL) {
                    // the exponential is masked, not the code: the row's factor
                    // may be 0 (a row of zeros quantised by its largest value),
                    // and -inf times it NaN
                    if (__builtin_amdgcn_ballot_w64(whole(j, ph[i])) != ~0ull) {
                        int lo, hi;
                        bounds(j, ph[i], lo, hi);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) x[e] = e >= lo && e < hi ? x[e] : 0.f;
                    }
                }
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    s += x[e];
                    if constexpr (BW) t = fmaf(x[e], g[e], t);
                    if constexpr (KEEP) ev[i][j * EPV + e] = x[e];
                }
                keep_order(s, t);
            }
            st[i][1] = wave_sum(s) * USH;
            if constexpr (BW) {
                t = wave_sum(t);
                if (SH != 0.f && __builtin_expect(!(fabsf(t) < INFINITY), 0)) {
                    // gradients from 2^96 on: the terms without their 2^32
                    t = 0.f;
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        if (empty(j, ph[i])) continue;
                        float g[EPV];
                        decode<DT>(x1[i][j], g, 1.f);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) t = fmaf(ev[KEEP ? i : 0][KEEP ? j * EPV + e : 0] * USH, g[e], t);
                    }
                    st[i][S::NS - 1] = wave_sum(t);
                } else {
                    st[i][S::NS - 1] = t * USH;
                }
            }
        }
        stream_reduce<OP, R, SPLIT>(st, a, row0, nr, c, lds, parity);
        if constexpr (!KEEP) fresh();
        if constexpr (KEEP && BW) {
#pragma unroll
            for (int i = 0; i < R; ++i) opaque<V>(x1[i]);
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float cmax = st[i][0], inv_s = 1.f / st[i][1];
            const float csh = !FP8 && far_ref(ct[i]) ? kExpShift + (ct[i] - cmax) : kExpShift - cmax, mul = inv_s * kExpUnshift;
            const float cdot = BW ? st[i][S::NS - 1] * inv_s : 0.f;
            float f = mul;
            // the clamps keep 0 times the factor 0 for a wave without a finite element
            if constexpr (FP8) {
                // the largest output is 2^0 / s: the codes are 448 2^(v - c)
                f = fast_exp2(fminf(ct[i] - cmax, 64.f)) * kFp8Max;
                if (c == 0 && tid == 0 && i < nr) a.so[row0 + i] = inv_s / kFp8Max;
            } else if constexpr (KEEP && SH == 0.f) {
                f = fast_exp2(fminf(ct[i] - cmax, 64.f)) * inv_s;
            } else if constexpr (KEEP) {
                // y = e 2^(ct - c + 32) 2^-64 / s.  A wave whose maximum lies far
                // below the row's takes the two factors one by one, so that
                // neither their product nor the result underflows early.
                const float f1 = fast_exp2(fminf(ct[i] - cmax + kExpShift, 64.f));
                f = mul * kExpUnshift;
                if (f1 < 1.f) {
#pragma unroll
                    for (int e = 0; e < V * EPV; ++e) ev[i][e] *= f1;
                } else {
                    f *= f1;
                }
            }
#pragma unroll
            for (int j = 0; j < V; ++j) {
                float q[EPV], y[EPV], g[EPV];
                if constexpr (!KEEP) decode<DT>(x0[i][j], q, 1.f);
                if constexpr (BW) decode<DT>(x1[i][j], g, 1.f);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float y0 = (KEEP ? ev[i][j * EPV + e] : fast_exp2(fmaf(q[e], kLog2e, csh))) * f;
                    y[e] = BW ? y0 * (g[e] - cdot) : y0;
                }
                store(row0 + i, i < nr, j, ph[i], encode<DT>(y, 1.f));
            }
        }
    }
}

// Waves per SIMD that the compiler is held to: the short BF16 rows (73 registers
// without, 72 with 7 waves; 12662 x 1040 25.8 and 20.4 us).
constexpr int stream_softmax_waves(int op, int dt, int v) {
    return op == OP_SOFTMAX_FWD && dt == DT_BF16 && v == 2 ? 7 : 4;
}

// FULL: every slice holds exactly V vectors per thread (N = k V T vectors).
template <int OP, int DT, int V, int R, bool SPLIT, bool FULL>
__global__ __launch_bounds__(64 * stream_max_waves(OP, DT, V, R))
__attribute__((amdgpu_waves_per_eu(SPLIT ? 4 : stream_softmax_waves(OP, DT, V)))) void k_stream_softmax(RowArgs a) {
    if (SPLIT && a.epoch == 0u && a.epoch_ptr)
        a.epoch = __hip_atomic_load(a.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __shared__ StreamLds<OP, R> lds;
    int c = 0, grp = blockIdx.x;
    if constexpr (SPLIT) member_of(a, blockIdx.x, c, grp);
    stream_softmax_rows<OP, DT, V, R, FULL, SPLIT>(a, c, grp, lds);
}

}  // namespace credit
