// stream_fp8.h -- the streaming form (stream.h) of the FP8 LayerNorm forward.
//
// The one-row kernel reads 8 bytes of gamma / beta for every byte of the row,
// twice per row: 4096 x 65536 moved 4.3 GB through the L2s for 0.5 GB of HBM
// traffic and took 2.6 times as long as the latter (220 us for 83).  Here a lane
// holds one vector (16 elements) of a slice with its gamma / beta in registers
// for all its rows, a round is 4 rows, and later rounds' loads are in flight:
// 140 us with k = 8.
//
// The statistics (mean and M2, then the largest output) of the rows are reduced
// for 4 rows at once: a wave folds its 4 registers into one, lane group ri (16
// lanes) holding row ri, so that merging waves, polling the members of a split
// row, the reciprocal square root and the output scale are one instruction for
// 4 rows.  On split rows the statistics of the next round travel with the
// largest output of this one, and the round before is written while they do:
// one exchange per round, none of it waited for (two, in sequence: 146 us with k
// = 4, 118 without waiting for the polls; 1024 x 262144 k
// = 16 166 -> 151).
//
// Bound: arithmetic, 12 instructions an element (90 of the 140 us: the output is
// evaluated once for its maximum and once to be written), and the next rows'
// loads, which have registers only from the moment the rows before are written.
// More does not fit: the outputs kept between the two take 64 registers of the
// 128 that 16 waves leave a lane (177-187 us with 8 waves), 8 rows a round spill.
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

// (count, mean, M2) and a maximum.
struct MergeChanMax {
    __device__ __forceinline__ void operator()(float (&a)[4], const float (&b)[4]) const {
        float x[3] = {a[0], a[1], a[2]};
        const float y[3] = {b[0], b[1], b[2]};
        MergeChanSel()(x, y);
        a[0] = x[0]; a[1] = x[1]; a[2] = x[2];
        a[3] = fmaxf(a[3], b[3]);
    }
};

struct StreamF8Lds {
    float red[2][kStreamWaves][kF8Rows][4];
    float xb[kF8Rows][4];
};

// Merges the waves' tuples, row i of the rounds in lane group i: (count, mean,
// M2) of the `ns` rows at `srow`, and the largest output of the `na` rows at `arow`.
// Row-resident: every wave gets the merged tuples.  Split: wave 0 does, and
// publishes them; f8_gather returns those of the row group.
template <bool SPLIT>
__device__ __forceinline__ void f8_publish(float (&v)[4], const RowArgs &a, int64_t srow, int ns, int64_t arow, int na,
                                           int c, StreamF8Lds &lds, int &parity) {
    constexpr int G = kF8Group;
    const MergeChanMax merge;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const int ri = fold_row(lane), p = lane & (G - 1);
    if (nw > 1) {
        float(*red)[kF8Rows][4] = lds.red[parity];
        if (p == 0) *(f32x4 *)red[wave][ri] = f32x4{v[0], v[1], v[2], v[3]};
        lds_barrier();
        parity ^= 1;
        if (!SPLIT || wave == 0) {
#pragma unroll
            for (int h = 0; h < kStreamWaves / G; ++h) {
                const int w = p + G * h;
                f32x4 u = {0.f, 0.f, 0.f, 0.f};
                if (w < nw) u = *(const f32x4 *)red[w][ri];
                const float o[4] = {u.x, u.y, u.z, u.w};
                if (h == 0) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) v[s] = o[s];
                } else {
                    merge(v, o);
                }
            }
            group_levels(v, merge);
        }
    }
    if constexpr (SPLIT) {
        if (a.flags & F_TEST_SKEW) {  // test only, as in device.h
            const uint64_t ticks = (uint64_t)((c * 7 + srow) % 13) * 100u;
            const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
            while (__builtin_amdgcn_s_memrealtime() - t0 < ticks) __builtin_amdgcn_s_sleep(8);
        }
        if (wave == 0 && p == 0 && !((a.flags & F_TEST_DROP_PUBLISH) && c == 1)) {
            auto publish = [&](unsigned long long *slot, float f) {
                __hip_atomic_store(slot, ((unsigned long long)a.epoch << 32) | __float_as_uint(f), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            };
            if (ri < ns) {
                publish(slot_ptr(a, srow + ri, 0, c, 0), v[1]);
                publish(slot_ptr(a, srow + ri, 0, c, 1), v[2]);
            }
            if (ri < na) publish(slot_ptr(a, arow + ri, 1, c, 0), v[3]);
        }
    }
}

// The row group's tuples of the rows that f8_publish named.  The count of a
// member follows from its slice.  Bounded waits as in device.h's exchange.
__device__ __forceinline__ void f8_gather(float (&v)[4], const RowArgs &a, int64_t srow, int ns, int64_t arow, int na,
                                          StreamF8Lds &lds) {
    constexpr int G = kF8Group;
    const MergeChanMax merge;
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // else what follows from it is kept in registers between calls
    const int ri = fold_row(lane), p = lane & (G - 1);
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) {
        constexpr int H = kMaxK / G;  // lane p of row ri polls members p, p + G, ...
        bool ok[H][3];
        float g[H][4];
        // (a row's slots: stages of k members of qs words)
        const char *sb = (const char *)slot_ptr(a, srow, 0, 0, 0), *ab = (const char *)slot_ptr(a, arow, 1, 0, 0);
        uint32_t at[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int m = p + G * h;
            const bool nos = m >= a.k || ri >= ns, noa = m >= a.k || ri >= na;
            at[h] = (uint32_t)((ri * kMaxStages * a.k + m) * a.qs * 8);
            ok[h][0] = ok[h][1] = nos;
            ok[h][2] = noa;
            const int64_t left = a.N - (int64_t)m * a.chunk;
            g[h][0] = nos || left <= 0 ? 0.f : (float)(left < a.chunk ? left : a.chunk);
            g[h][1] = g[h][2] = g[h][3] = 0.f;
        }
        unsigned spins = 0;
        while (true) {
            bool all = true;
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    if (!ok[h][x]) {
                        const unsigned long long w =
                            __hip_atomic_load((const unsigned long long *)((x < 2 ? sb + 8 * x : ab) + at[h]),
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        ok[h][x] = (unsigned)(w >> 32) == a.epoch;
                        if (ok[h][x]) g[h][x + 1] = __uint_as_float((unsigned)w);
                    }
                    all = all && ok[h][x];
                }
            if (__all(all)) break;
            if (++spins > a.spin_limit ||
                ((spins & 31u) == 0u &&
                 __hip_atomic_load(a.errflag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.epoch)) {
                if (lane == 0) __hip_atomic_store(a.errflag, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int h = 1; h < H; ++h) merge(g[0], g[h]);
        group_levels(g[0], merge);
        if (p == 0) *(f32x4 *)lds.xb[ri] = f32x4{g[0][0], g[0][1], g[0][2], g[0][3]};
    }
    lds_barrier();
    const f32x4 u = *(const f32x4 *)lds.xb[ri];
    v[0] = u.x; v[1] = u.y; v[2] = u.z; v[3] = u.w;
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
    const bool any = lane_full || lane_part;
    const int lo = lane_part ? 16 - tn : 0;  // first own element of the partial vector
    const bool wave_full = FULL || __builtin_amdgcn_ballot_w64(lane_full) == ~0ull;
    const bool wave_part = !FULL && __builtin_amdgcn_ballot_w64(lane_part) != 0;
    const float held = FULL ? 1024.f : wave_sum(lane_full ? 16.f : lane_part ? (float)tn : 0.f);
    const float inv_held = held > 0.f ? 1.f / held : 0.f;
    const int ri = fold_row(lane);
    const bool lead = c == 0 && tid < 64 && (lane & (kF8Group - 1)) == 0;

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

    struct Rows {
        u32x4 x[R];
        float xs;      // input scale of row ri
    };

    const int64_t step = (int64_t)a.groups * R;
    // The lane's row of a round, opaque: as an induction the compiler keeps a
    // 64-bit pointer per lane for each of the arrays indexed by it.
    auto here = [&]() -> uint32_t {
        uint32_t r = (uint32_t)ri;
        asm volatile("" : "+v"(r));
        return r;
    };
    // Loads of the rows at `row0`; past the end every lane reads the first
    // vector of the last rows again (one line).
    auto issue = [&](Rows &n, int64_t row0) {
        const bool live = row0 < a.M;
        const int64_t at = live ? row0 : a.M - 1;
        uint32_t o = live ? off : 0u;
        asm volatile("" : "+v"(o));
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t row = at + i < a.M ? at + i : at;
            n.x[i] = vload_nt<false>((const char *)a.in0 + row * a.ld0, o);
        }
        const int last = a.M - at > R ? R - 1 : (int)(a.M - at) - 1;
        const uint32_t rr = here();
        n.xs = (a.s0 + at)[(int)rr < last ? rr : (uint32_t)last];
    };
    auto count = [&](int64_t row0) -> int { return (int)(row0 >= a.M ? 0 : a.M - row0 < R ? a.M - row0 : R); };
    // (count, mean, M2) of the wave's part
    auto moments = [&](Rows &n, float (&st)[4]) {
        // Sum and sum of squares of the codes, two elements an instruction (an
        // e4m3 value is exact in FP16; products and sums are FP32).
        float s1[R], s2[R];
        if (!wave_full) {
            // codes that are not the lane's own count as 0
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int own = any ? 4 * w + 4 - lo : 0;  // bytes of this word, from its top
                const unsigned m = own >= 4 ? 0xffffffffu : own <= 0 ? 0u : 0xffffffffu << (8 * (4 - own));
#pragma unroll
                for (int i = 0; i < R; ++i) n.x[i][w] &= m;
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            s1[i] = s2[i] = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const unsigned d = n.x[i][w];
                const f16x2 one = {(_Float16)1.f, (_Float16)1.f};
                const f16x2 p = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(d, 1.f, false));
                const f16x2 q = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(d, 1.f, true));
                s1[i] = __builtin_amdgcn_fdot2(p, one, s1[i], false);
                s2[i] = __builtin_amdgcn_fdot2(p, p, s2[i], false);
                s1[i] = __builtin_amdgcn_fdot2(q, one, s1[i], false);
                s2[i] = __builtin_amdgcn_fdot2(q, q, s2[i], false);
            }
            keep_order(s1[i], s2[i]);
        }
        const float mw = fold(s1, FoldSum()) * inv_held;
        float m2 = fold(s2, FoldSum()) - held * mw * mw, mean = mw;
        // Where the mean is large beside the spread the difference of the two
        // has lost digits: moments about the wave's mean instead, for those rows
        // (a row's result is not to depend on the others of its round).
        const bool lost = !(held * mw * mw <= 2.f * m2);
        if (__builtin_amdgcn_ballot_w64(lost) != 0) {
            opaque<R>(n.x);
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const float m = lane_value(mw, fold_lane(i));
                float q[16];
                s1[i] = s2[i] = 0.f;
                decode<DT_FP8>(n.x[i], q, 1.f);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float d = any && e >= lo ? q[e] - m : 0.f;
                    s1[i] += d;
                    s2[i] = fmaf(d, d, s2[i]);
                }
                keep_order(s1[i], s2[i]);
            }
            const float f1 = fold(s1, FoldSum()), f2 = fold(s2, FoldSum()), r = f1 * inv_held;
            mean = lost ? mean + r : mean;
            m2 = lost ? f2 - f1 * r : m2;
        }
        st[0] = held;
        st[1] = held > 0.f ? mean : 0.f;
        st[2] = held > 0.f && !(m2 < 0.f) ? m2 : 0.f;  // NaN stays (stream.h)
    };
    // the scales by which rows are written: with the largest output `am`, 448 / am
    struct Out {
        float amul, bm, oinv;
        bool plain;
        uint64_t cent;  // by lane
    };
    // y = (q amul + bm) gamma + beta with bm = -mean amul, whose rounding is below
    // those of q - mean and its product while |bm| is small.  A row whose mean lies
    // half a spread or more from 0 (a constant row has no spread: a rounding of
    // 448 / sqrt(eps) would be its output) has its `cent` bit set and bm the mean: y
    // = (q - bm) amul gamma + beta, one instruction an element more (calls of 4096 x
    // 65536, k = 8: 154 -> 159 us, 185 -> 199 where every row is such a one; 168 with
    // the instruction in every row).
    auto finish = [&](const Rows &n, const float (&st)[4], int64_t row0, Out &o) {
        const float mean = st[1], rstd = rsqrtf(n.xs * n.xs * (st[2] * invN) + a.eps);
        o.amul = n.xs * rstd;
        o.bm = -mean * o.amul;
        const bool cent = !(fabsf(o.bm) <= 0.5f);
        o.cent = __builtin_amdgcn_ballot_w64(cent);
        o.bm = cent ? mean : o.bm;
        if (lead && row0 + ri < a.M) {
            const uint32_t rr = here();
            if (a.mean_out) (a.mean_out + row0)[rr] = n.xs * mean;
            if (a.rstd_out) (a.rstd_out + row0)[rr] = rstd;
        }
    };
    // decoded codes of row i -> y
    auto output = [&](float (&q)[16], const Out &o, int i) {
        const float A = lane_value(o.amul, fold_lane(i));
        float Bm = lane_value(o.bm, fold_lane(i));
        if (o.cent >> fold_lane(i) & 1) {
#pragma unroll
            for (int e = 0; e < 16; ++e) q[e] -= Bm;
            Bm = 0.f;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) q[e] = fmaf(fmaf(q[e], A, Bm), g[e], b[e]);
    };
    auto largest = [&](Rows &cur, const Out &o) -> float {
        float t[R];
        opaque<R>(cur.x);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            float q[16], am = 0.f;
            decode<DT_FP8>(cur.x[i], q, 1.f);
            output(q, o, i);
            if (wave_part) {
#pragma unroll
                for (int e = 0; e < 16; ++e) am = fmaxf(am, e >= lo ? fabsf(q[e]) : 0.f);
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) am = fmaxf(am, fabsf(q[e]));
            }
            t[i] = any ? am : 0.f;
            keep_order(t[i]);
        }
        return fold(t, FoldMax());
    };
    auto write = [&](Rows &cur, const Out &o, int64_t row0) {
        const int nr = count(row0);
        uint32_t so = off;
        asm volatile("" : "+v"(so));
        opaque<R>(cur.x);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float oi = lane_value(o.oinv, fold_lane(i));
            float q[16];
            decode<DT_FP8>(cur.x[i], q, 1.f);
            output(q, o, i);
            u32x4 v;
            if (o.plain) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    int d = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * w] * oi, q[4 * w + 1] * oi, 0, false);
                    v[w] = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(q[4 * w + 2] * oi, q[4 * w + 3] * oi, d, true);
                }
            } else {
                v = encode<DT_FP8>(q, oi);
            }
            // unconditional, dropped for lanes without a whole vector (stream.h)
            char *orow = (char *)a.out + (row0 + i) * a.ldo;
            __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(orow, 0, i < nr ? (int)a.N : 0, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, lane_full ? so : 0x80000000u, 0, CREDIT_STORE_NT ? 2 : 0);
            if (!FULL && i < nr && lane_part) {
#pragma unroll
                for (int e = 1; e < 16; ++e)
                    if (e >= lo) (orow + so)[e] = (char)(v[e / 4] >> (8 * (e & 3)));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto scale = [&](Out &o, float am, int64_t row0) {
        o.oinv = am > 0.f ? kFp8Max / am : 1.f;
        if (lead && row0 + ri < a.M) (a.so + row0)[here()] = am > 0.f ? am / kFp8Max : 1.f;
        // Finite rows scaled by 448 / amax convert without a clamp (up to 464
        // rounds to 448); anything else takes the clamp, so do rows so small that
        // 448 / amax is infinite.
        o.plain = pfin && __builtin_amdgcn_ballot_w64(fabsf(o.amul) < 1e30f && fabsf(o.bm) < 1e30f && am < 3e38f &&
                                                      o.oinv < 3e38f) == ~0ull;
    };

    // A round: the largest output of the current rows and the moments of the
    // next ones are published; the rows before, whose scale is known, are
    // written while that is under way, the rows move up and the loads of the
    // rows after the next are issued; then the row group's values are gathered.
    // Wave 0, which polls, loads after that: loads return in order.
    const bool poller = T > 64 && __builtin_amdgcn_readfirstlane(tid >> 6) == 0;
    int64_t row0 = (int64_t)grp * R;
    if (row0 >= a.M) return;
    Rows prv, cur, nxt;
    Out oc, op;  // of the current and the previous rows
    float st[4];
    if constexpr (!SPLIT) {
        // Row-resident: nothing to wait for but a barrier, so two sets of rows
        // do (4096 x 16384: 32.7 us, 37.6 with three); rows off their lines take
        // longer to load, so theirs are issued first.
        issue(nxt, row0);
        __builtin_amdgcn_s_waitcnt(0);  // the loop's own waits then count its own accesses only
        for (; row0 < a.M; row0 += step) {
            cur = nxt;
            if (!FULL) issue(nxt, row0 + step);
            __builtin_amdgcn_sched_barrier(0);
            moments(cur, st);
            st[3] = 0.f;
            f8_publish<SPLIT>(st, a, row0, 0, row0, 0, c, lds, parity);
            finish(cur, st, row0, oc);
            if (FULL) issue(nxt, row0 + step);
            const float fm = largest(cur, oc);
            st[0] = st[1] = st[2] = 0.f;
            st[3] = fm;
            f8_publish<SPLIT>(st, a, row0, 0, row0, 0, c, lds, parity);
            scale(oc, st[3], row0);
            write(cur, oc, row0);
        }
        return;
    }
    issue(cur, row0);
    issue(nxt, row0 + step);
    moments(cur, st);
    st[3] = 0.f;
    f8_publish<SPLIT>(st, a, row0, count(row0), row0, 0, c, lds, parity);
    f8_gather(st, a, row0, count(row0), row0, 0, lds);
    finish(cur, st, row0, oc);
    op = oc;
    op.oinv = 0.f;
    op.plain = false;
    prv = cur;
    __builtin_amdgcn_s_waitcnt(0);  // the loop's own waits then count its own accesses only
    bool first = true;
    for (; row0 < a.M; row0 += step) {
        const int nr = count(row0), nn = count(row0 + step);
        const float fm = largest(cur, oc);
        moments(nxt, st);
        st[3] = fm;
        f8_publish<SPLIT>(st, a, row0 + step, nn, row0, nr, c, lds, parity);
        if (!first) write(prv, op, row0 - step);
        first = false;
        // (made here, so that the loads go to the registers they leave)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            prv.x[i] = cur.x[i];
            cur.x[i] = nxt.x[i];
        }
        opaque<R>(prv.x);
        opaque<R>(cur.x);
        cur.xs = nxt.xs;
        keep1(cur.xs);
        if (!poller) issue(nxt, row0 + 2 * step);
        f8_gather(st, a, row0 + step, nn, row0, nr, lds);
        if (poller) issue(nxt, row0 + 2 * step);
        scale(oc, st[3], row0);
        op = oc;
        finish(cur, st, row0 + step, oc);
    }
    write(prv, op, row0 - step);
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
