// stream_fp8.h -- the streaming form (stream.h) of the FP8 LayerNorm forward.
//
// The one-row kernel reads 8 bytes of gamma / beta for every byte of the row,
// twice per row: 4096 x 65536 moved 4.3 GB through the L2s for 0.5 GB of HBM
// traffic and took 2.6 times as long as the latter (220 us for 83).  Here a lane
// holds one vector (16 elements) of a slice with its gamma / beta in registers
// for all its rows, a round is 4 rows, and the next round's loads are in flight:
// 146 us with k = 4.
//
// The statistics of a round's rows are reduced for all of them at once: a wave
// folds its 4 registers into one, lane group ri (16 lanes) holding row ri, so that merging waves, polling the members of a split row, the reciprocal
// square root and the output scale are one instruction for 4 rows.
//
// Bound: arithmetic, 12 instructions an element (90 of the 146 us: the output is
// evaluated once for its maximum and once to be written), and the two exchanges
// of a round (28 us).  More does not fit: the outputs kept between the two take
// 64 registers of the 128 that 16 waves leave a lane (177-187 us with 8), 8 rows
// a round spill (153), and moving the next round's statistics into the exchange
// of this one's maximum, with three sets of rows, spills as well (143-147; 35
// against 33 us where nothing is exchanged, 4096 x 16384).
#pragma once
#include "stream.h"

namespace credit {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kF8Rows = 4;             // rows of a round
constexpr int kF8Group = 64 / kF8Rows;  // lanes of a group

// Lane of the wave from which row i's folded value is taken, and the row a
// lane's group holds.
constexpr int fold_lane(int i) { return (i >> 1) * 32 + (i & 1) * 16; }
__device__ __forceinline__ int fold_row(int lane) { return ((lane >> 5) & 1) * 2 + ((lane >> 4) & 1); }
// Over the lanes of a group (all of them get the result).
template <int NV, class F> __device__ __forceinline__ void group_levels(float (&v)[NV], F f) {
    float o[NV];
#define CREDIT_LEVEL(CTRL)                                                              \
    _Pragma("unroll") for (int i = 0; i < NV; ++i) o[i] = dpp_or<CTRL, 0xF>(v[i], v[i]); \
    f(v, o);
    CREDIT_LEVEL(0xB1)   // lane ^ 1
    CREDIT_LEVEL(0x4E)   // lane ^ 2
    CREDIT_LEVEL(0x141)  // mirrored in 8
    CREDIT_LEVEL(0x140)  // mirrored in 16
#undef CREDIT_LEVEL
}
struct FoldSum {
    __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct FoldMax {
    __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
// One value per lane and row -> one: row fold_row(lane)'s, over the wave's lanes.
template <class F> __device__ __forceinline__ float fold(const float (&v)[kF8Rows], F f) {
    float a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 2]), false, false);
        a[i] = f(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[0]), __float_as_uint(a[1]), false, false);
    float c[1] = {f(__uint_as_float(r[0]), __uint_as_float(r[1]))};
    group_levels(c, [&](float (&x)[1], const float (&o)[1]) { x[0] = f(x[0], o[0]); });
    return c[0];
}

// (count, mean, M2) or a single maximum, in lane groups: merge rules.
struct MergeMax1 {
    __device__ __forceinline__ void operator()(float (&a)[1], const float (&b)[1]) const { a[0] = fmaxf(a[0], b[0]); }
};

struct StreamF8Lds {
    float red[2][kStreamWaves][kF8Rows][3];
    float xb[kF8Rows][3];
};

// Merges the waves' (and members') tuples of the rows, one row per lane group;
// STAGE 0: (count, mean, M2), the count of a member following from its slice;
// STAGE 1: the largest output.  As stream_reduce otherwise.
template <bool SPLIT, int STAGE, int NS, class Merge>
__device__ __forceinline__ void f8_reduce(float (&v)[NS], Merge merge, const RowArgs &a, int64_t row0, int nr, int c,
                                          StreamF8Lds &lds, int &parity) {
    constexpr int G = kF8Group, NX = STAGE == 0 ? 2 : 1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const int ri = fold_row(lane), p = lane & (G - 1);
    if (nw > 1) {
        float(*red)[kF8Rows][3] = lds.red[parity];
        if (p == 0) {
#pragma unroll
            for (int s = 0; s < NS; ++s) red[wave][ri][s] = v[s];
        }
        lds_barrier();
        parity ^= 1;
        if (!SPLIT || wave == 0) {
#pragma unroll
            for (int h = 0; h < kStreamWaves / G; ++h) {
                float o[NS];
#pragma unroll
                for (int s = 0; s < NS; ++s) o[s] = p + G * h < nw ? red[p + G * h][ri][s] : 0.f;
                if (h == 0) {
#pragma unroll
                    for (int s = 0; s < NS; ++s) v[s] = o[s];
                } else {
                    merge(v, o);
                }
            }
            group_levels(v, merge);
        }
    }
    if constexpr (SPLIT) {
        if (a.flags & F_TEST_SKEW) {  // test only, as in device.h
            const uint64_t ticks = (uint64_t)((c * 7 + row0 + STAGE) % 13) * 100u;
            const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
            while (__builtin_amdgcn_s_memrealtime() - t0 < ticks) __builtin_amdgcn_s_sleep(8);
        }
        if (wave == 0) {
            if (p == 0 && ri < nr && !((a.flags & F_TEST_DROP_PUBLISH) && c == 1)) {
#pragma unroll
                for (int x = 0; x < NX; ++x) {
                    const float pv = v[NS - NX + x];
                    __hip_atomic_store(slot_ptr(a, row0 + ri, STAGE, c, x),
                                       ((unsigned long long)a.epoch << 32) | __float_as_uint(pv), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            constexpr int H = kMaxK / G;  // lane p of row ri polls members p, p + G, ...
            bool ok[H][NX];
            float g[H][NS];
            const char *base = (const char *)slot_ptr(a, row0, STAGE, 0, 0);
            uint32_t at[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int m = p + G * h;
                const bool none = m >= a.k || ri >= nr;
                at[h] = (uint32_t)((ri * kMaxStages * a.k + m) * a.qs * 8);
#pragma unroll
                for (int x = 0; x < NX; ++x) ok[h][x] = none;
#pragma unroll
                for (int s = 0; s < NS; ++s) g[h][s] = 0.f;
                if constexpr (STAGE == 0) {
                    const int64_t left = a.N - (int64_t)m * a.chunk;
                    g[h][0] = none || left <= 0 ? 0.f : (float)(left < a.chunk ? left : a.chunk);
                }
            }
            unsigned spins = 0;
            while (true) {
                bool all = true;
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        if (!ok[h][x]) {
                            const unsigned long long w =
                                __hip_atomic_load((const unsigned long long *)(base + at[h] + 8 * x), __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                            ok[h][x] = (unsigned)(w >> 32) == a.epoch;
                            if (ok[h][x]) g[h][NS - NX + x] = __uint_as_float((unsigned)w);
                        }
                        all = all && ok[h][x];
                    }
                if (__all(all)) break;
                if (++spins > a.spin_limit ||
                    ((spins & 31u) == 0u &&
                     __hip_atomic_load(a.errflag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.epoch)) {
                    if (lane == 0)
                        __hip_atomic_store(a.errflag, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (int h = 1; h < H; ++h) merge(g[0], g[h]);
            group_levels(g[0], merge);
            if (p == 0) {
#pragma unroll
                for (int s = 0; s < NS; ++s) lds.xb[ri][s] = g[0][s];
            }
        }
        lds_barrier();
#pragma unroll
        for (int s = 0; s < NS; ++s) v[s] = lds.xb[ri][s];
    }
}

template <bool SPLIT, bool FULL>
__device__ __forceinline__ void stream_ln_fp8_rows(const RowArgs &a, int c, int grp, StreamF8Lds &lds) {
    constexpr int R = kF8Rows;
    const int tid = threadIdx.x, lane = tid & 63, T = (int)blockDim.x;
    int parity = 0;
    const float invN = 1.f / (float)a.N;
    // the slice (as in stream.h, one slot)
    const int64_t c0 = (int64_t)c * a.chunk;
    const int64_t left = a.N - c0;
    const int nval = (int)(left <= 0 ? 0 : left < a.chunk ? left : a.chunk);
    const int nfv = nval / 16, tn = nval - nfv * 16;
    const uint32_t rowlast = (uint32_t)a.N - 16u;
    uint32_t off = (uint32_t)c0 + (uint32_t)tid * 16u;
    if (!FULL) off = off < rowlast ? off : rowlast;
    const bool lane_full = FULL || tid < nfv, lane_part = !FULL && tid == nfv && tn > 0;
    const int lo = lane_part ? 16 - tn : 0;  // first own element of the partial vector
    const bool any = lane_full || lane_part;
    const bool wave_full = FULL || __builtin_amdgcn_ballot_w64(lane_full) == ~0ull;
    const bool wave_part = !FULL && __builtin_amdgcn_ballot_w64(lane_part) != 0;
    const float held = FULL ? 1024.f : wave_sum(lane_full ? 16.f : lane_part ? (float)tn : 0.f);
    const float inv_held = held > 0.f ? 1.f / held : 0.f;
    const int ri = fold_row(lane);
    const bool lead = (lane & (kF8Group - 1)) == 0;

    float g[16], b[16];
    bool fin = true;
#pragma unroll
    for (int i = 0; i < 16; i += 4) {
        const f32x4 u = *(const f32x4_u *)(a.gamma + off + i), w = *(const f32x4_u *)(a.beta + off + i);
        g[i] = u.x; g[i + 1] = u.y; g[i + 2] = u.z; g[i + 3] = u.w;
        b[i] = w.x; b[i + 1] = w.y; b[i + 2] = w.z; b[i + 3] = w.w;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) fin = fin && __builtin_isfinite(g[i]) && __builtin_isfinite(b[i]);
    const bool pfin = __builtin_amdgcn_ballot_w64(fin) == ~0ull;

    // The lane's row of a round, opaque: as an induction the compiler keeps a
    // 64-bit pointer per lane for each of the arrays indexed by it.
    auto here = [&]() -> uint32_t {
        uint32_t r = (uint32_t)ri;
        asm volatile("" : "+v"(r));
        return r;
    };
    u32x4 x[R], n[R];
    float xs, nxs;          // input scale of row ri
    auto issue = [&](int64_t row0, uint32_t live) {
        uint32_t o = off & live;
        asm volatile("" : "+v"(o));
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t row = row0 + i < a.M ? row0 + i : row0;
            n[i] = vload_nt<false>((const char *)a.in0 + row * a.ld0, o);
        }
        const int last = a.M - row0 > R ? R - 1 : (int)(a.M - row0) - 1;
        const uint32_t rr = here();
        nxs = (a.s0 + row0)[(int)rr < last ? rr : (uint32_t)last];
    };
    uint32_t so;
    auto store = [&](int64_t row, bool live, u32x4 v) {
        char *orow = (char *)a.out + row * a.ldo;
        __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(orow, 0, live ? (int)a.N : 0, 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b128(v, rs, lane_full ? so : 0x80000000u, 0, CREDIT_STORE_NT ? 2 : 0);
        if (!FULL && live && lane_part) {
#pragma unroll
            for (int i = 1; i < 16; ++i)
                if (i >= lo) (orow + so)[i] = (char)(v[i / 4] >> (8 * (i & 3)));
        }
    };

    const int64_t step = (int64_t)a.groups * R;
    int64_t row0 = (int64_t)grp * R;
    if (row0 < a.M) issue(row0, 0xffffffffu);
    __builtin_amdgcn_s_waitcnt(0);  // the loop's own waits then count its own accesses only
    for (; row0 < a.M; row0 += step) {
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = n[i];
        xs = nxs;
        const int64_t nrow = row0 + step;
        // (rows off their lines take longer to load: theirs go first)
        constexpr bool EARLY = !FULL;
        const bool poller = SPLIT && T > 64 && __builtin_amdgcn_readfirstlane(tid >> 6) == 0;
        auto next = [&]() { issue(nrow < a.M ? nrow : row0, nrow < a.M ? 0xffffffffu : 0u); };
        if (EARLY && !poller) next();
        __builtin_amdgcn_sched_barrier(0);
        const int nr = (int)(a.M - row0 < R ? a.M - row0 : R);
        so = off;
        asm volatile("" : "+v"(so));
        const bool writer = c == 0 && tid < 64 && lead && ri < nr;
        // Sum and sum of squares of the codes, two elements an instruction (an
        // e4m3 value is exact in FP16; products and sums are FP32), then (count,
        // mean, M2) of the wave.
        float s1[R], s2[R];
        if (!wave_full) {
            // codes that are not the lane's own count as 0
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int own = any ? 4 * w + 4 - lo : 0;  // bytes of this word, from its top
                const unsigned m = own >= 4 ? 0xffffffffu : own <= 0 ? 0u : 0xffffffffu << (8 * (4 - own));
#pragma unroll
                for (int i = 0; i < R; ++i) x[i][w] &= m;
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            s1[i] = s2[i] = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const unsigned d = x[i][w];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const f16x2 q = __builtin_bit_cast(f16x2, u ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(d, 1.f, true)
                                                                : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(d, 1.f, false));
                    s1[i] = __builtin_amdgcn_fdot2(q, f16x2{(_Float16)1.f, (_Float16)1.f}, s1[i], false);
                    s2[i] = __builtin_amdgcn_fdot2(q, q, s2[i], false);
                }
            }
            keep_order(s1[i], s2[i]);
        }
        const float mw = fold(s1, FoldSum()) * inv_held;
        float m2 = fold(s2, FoldSum()) - held * mw * mw, mean_w = mw;
        // Where the mean is large beside the spread the difference of the two
        // has lost digits: moments about the wave's mean instead.
        if (__builtin_amdgcn_ballot_w64(!(held * mw * mw <= 2.f * m2)) != 0) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const float m = lane_value(mw, fold_lane(i));
                float q[16];
                s1[i] = s2[i] = 0.f;
                decode<DT_FP8>(x[i], q, 1.f);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float d = any && e >= lo ? q[e] - m : 0.f;
                    s1[i] += d;
                    s2[i] = fmaf(d, d, s2[i]);
                }
                keep_order(s1[i], s2[i]);
            }
            const float f1 = fold(s1, FoldSum()), f2 = fold(s2, FoldSum()), r = f1 * inv_held;
            mean_w += r;
            m2 = f2 - f1 * r;
        }
        float st[3] = {held, held > 0.f ? mean_w : 0.f, held > 0.f ? fmaxf(m2, 0.f) : 0.f};
        f8_reduce<SPLIT, 0, 3>(st, MergeChanSel(), a, row0, nr, c, lds, parity);
        if (!EARLY && !poller) next();
        const float mean = st[1], rstd = rsqrtf(xs * xs * (st[2] * invN) + a.eps);
        const float amul = xs * rstd, bm = -mean * amul;
        if (writer) {
            const uint32_t rr = here();
            if (a.mean_out) (a.mean_out + row0)[rr] = xs * mean;
            if (a.rstd_out) (a.rstd_out + row0)[rr] = rstd;
        }
        opaque<R>(x);
        float t[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float A = lane_value(amul, fold_lane(i)), Bm = lane_value(bm, fold_lane(i));
            float q[16], am = 0.f;
            decode<DT_FP8>(x[i], q, 1.f);
            if (wave_part) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float y = fmaf(fmaf(q[e], A, Bm), g[e], b[e]);
                    am = fmaxf(am, e >= lo ? fabsf(y) : 0.f);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) am = fmaxf(am, fabsf(fmaf(fmaf(q[e], A, Bm), g[e], b[e])));
            }
            if (!FULL) am = any ? am : 0.f;
            t[i] = am;
            keep_order(t[i]);
        }
        float mx[1] = {fold(t, FoldMax())};
        f8_reduce<SPLIT, 1, 1>(mx, MergeMax1(), a, row0, nr, c, lds, parity);
        if (poller) next();
        const float oinv = mx[0] > 0.f ? kFp8Max / mx[0] : 1.f;
        if (writer) (a.so + row0)[here()] = mx[0] > 0.f ? mx[0] / kFp8Max : 1.f;
        // Finite rows scaled by 448 / amax convert without a clamp (up to 464
        // rounds to 448); anything else takes the clamp.
        const bool plain = pfin && __builtin_amdgcn_ballot_w64(fabsf(amul) < 1e30f && fabsf(bm) < 1e30f &&
                                                               mx[0] < 3e38f) == ~0ull;
        opaque<R>(x);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float A = lane_value(amul, fold_lane(i)), Bm = lane_value(bm, fold_lane(i));
            const float oi = lane_value(oinv, fold_lane(i));
            float q[16];
            decode<DT_FP8>(x[i], q, 1.f);
#pragma unroll
            for (int e = 0; e < 16; ++e) q[e] = fmaf(fmaf(q[e], A, Bm), g[e], b[e]);
            u32x4 v;
            if (plain) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    int d = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * w] * oi, q[4 * w + 1] * oi, 0, false);
                    v[w] = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(q[4 * w + 2] * oi, q[4 * w + 3] * oi, d, true);
                }
            } else {
                v = encode<DT_FP8>(q, oi);
            }
            store(row0 + i, i < nr, v);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// FULL: every slice is one whole vector per thread (N = 16 k T).
template <bool SPLIT, bool FULL>
__global__ __launch_bounds__(1024) void k_stream_ln_fp8(RowArgs a) {
    if (SPLIT && a.epoch == 0u && a.epoch_ptr)
        a.epoch = __hip_atomic_load(a.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __shared__ StreamF8Lds lds;
    int c = 0, grp = blockIdx.x;
    if constexpr (SPLIT) member_of(a, blockIdx.x, c, grp);
    stream_ln_fp8_rows<SPLIT, FULL>(a, c, grp, lds);
}

}  // namespace credit
