// stream.h -- the streaming form of the row-resident / split-row kernels: a
// workgroup keeps what is common to its rows (the gamma / beta slice, the
// dgamma / dbeta column sums) in registers for all of them, and has the next
// rows' loads in flight while it works on the current ones.
//
// The one-row kernels (resident.h) hold one row slice at a time: a workgroup
// loads, waits, reduces, exchanges, writes, and its memory pipe is idle from
// its last load's arrival to its first store.  What hides that is other
// workgroups, so those kernels are bound by occupancy wherever the slice is
// short or the register demand high (LayerNorm / RMSNorm backward), and by
// one gamma / beta read per row.  Here a round is R rows of the slice, and the
// loads of round i + 1 are issued before round i's arithmetic.
//
// A slice of nvec 16-byte vectors is held by w waves, V vectors a lane
// (w = ceil(nvec / 64 V), any w up to the instance's limit, so few lanes are
// idle whatever the width): vector j T + t of the slice is slot j of thread t
// of T = 64 w.  Rows of any width and alignment take the same 128-bit
// accesses; the partial vector at the end of a row is loaded as the last 16
// bytes of the row, with the elements that belong to its neighbour masked, so
// no load is done element by element (N is at least one vector).
//
// Statistics: each wave reduces its lanes with DPP and, alone in its
// workgroup, needs no barrier at all; else the waves' tuples go through LDS
// (one barrier per stage) and every wave merges them in its lanes, lane
// u R + i holding wave u of row i.  The split form publishes and polls R rows
// at a time, in wave 0 (the slots are those of the one-row kernels), and
// merges the members in its lanes in the same way.
//
// Bound: HBM where the rows are long enough (BF16 RMSNorm forward 8192 x 4096 and
// backward 8192 x 8192: 5.4 TB/s of 6.45); the exchange, whose polls return in
// order behind the next round's loads, on split rows (backward 2048 x 131072 k = 16:
// 4.7-5.3 TB/s); the column sums' partial rows on narrow ones of the backward;
// arithmetic and the launch on the forward's shortest (16384 x 1024 13.7 us for a
// floor of 10.4).  Before and after at each rule in host.cpp.
#pragma once
#include "resident.h"

namespace credit {

// Workgroup barrier that orders LDS only: global loads and stores in flight
// stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ------------------------------------------------------- lane reductions
template <int CTRL, int ROWS> __device__ __forceinline__ float dpp_or(float ident, float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(ident), __float_as_int(v), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
// Sum and maximum over the wave's 64 lanes (row_shr 1, 2, 4, 8, then the row
// broadcasts; lane 63 holds the result), uniform.
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_or<0x111, 0xF>(0.f, v);
    v += dpp_or<0x112, 0xF>(0.f, v);
    v += dpp_or<0x114, 0xF>(0.f, v);
    v += dpp_or<0x118, 0xF>(0.f, v);
    v += dpp_or<0x142, 0xA>(0.f, v);
    v += dpp_or<0x143, 0xC>(0.f, v);
    return lane_value(v, 63);
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_or<0x111, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_or<0x112, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_or<0x114, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_or<0x118, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_or<0x142, 0xA>(-INFINITY, v));
    v = fmaxf(v, dpp_or<0x143, 0xC>(-INFINITY, v));
    return lane_value(v, 63);
}
// Merges the tuples of lanes l, l + S, l + 2 S, ... of the wave (S = 1, 2 or
// 4; lanes past the last tuple hold the identity), `count` lanes in all:
// rotations inside the 16-lane rows, then the row exchanges.
template <int S, int NV, class Merge> __device__ __forceinline__ void lanes_merge(float (&v)[NV], int count, Merge merge) {
#define CREDIT_ROR(N)                                                                     \
    if constexpr (N >= S) {                                                               \
        float o[NV];                                                                      \
        _Pragma("unroll") for (int i = 0; i < NV; ++i) o[i] = dpp_or<0x120 + N, 0xF>(v[i], v[i]); \
        merge(v, o);                                                                      \
    }
    CREDIT_ROR(8)
    CREDIT_ROR(4)
    CREDIT_ROR(2)
    CREDIT_ROR(1)
#undef CREDIT_ROR
    if (count > 16) {
        float a[NV], b[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i]), false, false);
            a[i] = __uint_as_float(r[0]);
            b[i] = __uint_as_float(r[1]);
        }
        merge(a, b);
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = a[i];
    }
    if (count > 32) {
        float a[NV], b[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i]), false, false);
            a[i] = __uint_as_float(r[0]);
            b[i] = __uint_as_float(r[1]);
        }
        merge(a, b);
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = a[i];
    }
}

// (count, mean, M2) pairs, free of branches (lanes hold empty tuples).
struct MergeChanSel {
    __device__ __forceinline__ void operator()(float (&a)[3], const float (&b)[3]) const {
        const float n = a[0] + b[0], d = b[1] - a[1];
        const float w = a[0] == 0.f ? 1.f : b[0] == 0.f ? 0.f : b[0] * __builtin_amdgcn_rcpf(n);
        a[1] = a[0] == 0.f ? b[1] : b[0] == 0.f ? a[1] : a[1] + d * w;
        a[2] = a[0] == 0.f ? b[2] : b[0] == 0.f ? a[2] : a[2] + b[2] + d * d * a[0] * w;
        a[0] = n;
    }
};

// The statistics of an operator: per-wave tuple size, exchanged words, merge.
template <int OP> struct StreamStat {
    typedef MergeSum M;
    static constexpr int NS = 1, NX = 1;
    static constexpr float ident = 0.f;
};
template <> struct StreamStat<OP_LN_BWD> {
    typedef MergeSum M;
    static constexpr int NS = 2, NX = 2;
    static constexpr float ident = 0.f;
};
template <> struct StreamStat<OP_LN_FWD> {  // (count, mean about the row's first element, M2)
    typedef MergeChanSel M;
    static constexpr int NS = 3, NX = 2;
    static constexpr float ident = 0.f;
};
template <> struct StreamStat<OP_SOFTMAX_FWD> {
    typedef MergeSoftmax M;
    static constexpr int NS = 2, NX = 2;
    static constexpr float ident = -INFINITY;  // of the maximum
};
template <> struct StreamStat<OP_SMXL_BWD> {
    typedef MergeSoftmax3 M;
    static constexpr int NS = 3, NX = 3;
    static constexpr float ident = -INFINITY;
};

// LDS of a workgroup: the waves' tuples (two stages' worth, used in turn) and
// the merged tuples of the split form.
template <int OP, int R> struct StreamLds {
    float red[2][kStreamWaves * R][StreamStat<OP>::NS];
    float xb[R][StreamStat<OP>::NS];
};

// Merges R per-wave tuples (uniform in each wave) over the workgroup and, in
// the split form, over the row group; returns uniform tuples.  Bounded waits
// as in device.h's exchange; `blk` is the round's first row.
template <int OP, int R, bool SPLIT>
__device__ __forceinline__ void stream_reduce(float (&st)[R][StreamStat<OP>::NS], const RowArgs &a, int64_t row0, int nr,
                                              int c, StreamLds<OP, R> &lds, int &parity) {
    typedef StreamStat<OP> S;
    constexpr int NS = S::NS, NX = S::NX;
    typename S::M merge;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    if (nw == 1 && !SPLIT) return;
    float v[NS];
    if (nw > 1) {
        float(*red)[NS] = lds.red[parity];
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    float t = st[i][s];
                    keep1(t);  // else the copy is taken for a memcpy and st is put in memory
                    red[wave * R + i][s] = t;
                }
        }
        lds_barrier();
        parity ^= 1;
        if (!SPLIT || wave == 0) {
#pragma unroll
            for (int s = 0; s < NS; ++s) v[s] = s == 0 ? S::ident : 0.f;
            if (lane < nw * R) {
#pragma unroll
                for (int s = 0; s < NS; ++s) v[s] = red[lane][s];
            }
            lanes_merge<R, NS>(v, nw * R, merge);
        }
    } else if constexpr (SPLIT) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            v[s] = st[0][s];
#pragma unroll
            for (int i = 1; i < R; ++i) {
                float t = st[i][s];
                keep1(t);
                v[s] = lane == i ? t : v[s];
            }
        }
    }
    if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int s = 0; s < NS; ++s) st[i][s] = lane_value(v[s], i);
    } else {
        if (a.flags & F_TEST_SKEW) {  // test only, as in device.h
            const uint64_t ticks = (uint64_t)((c * 7 + row0) % 13) * 100u;
            const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
            while (__builtin_amdgcn_s_memrealtime() - t0 < ticks) __builtin_amdgcn_s_sleep(8);
        }
        if (wave == 0) {
            if (lane < nr && !((a.flags & F_TEST_DROP_PUBLISH) && c == 1)) {
#pragma unroll
                for (int x = 0; x < NX; ++x) {
                    const float pv = v[NS - NX + x];
                    __hip_atomic_store(slot_ptr(a, row0 + lane, 0, c, x),
                                       ((unsigned long long)a.epoch << 32) | __float_as_uint(pv), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            // lane l of half h polls member (l + 64 h) / R of row (l + 64 h) % R
            constexpr int H = (kMaxK * R + 63) / 64;
            bool ok[H][NX];
            float g[H][NS];
            const unsigned long long *p[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int e = lane + 64 * h, m = e / R, i = e % R;
                const bool none = m >= a.k || i >= nr;
                p[h] = none ? nullptr : slot_ptr(a, row0 + i, 0, m, 0);
#pragma unroll
                for (int x = 0; x < NX; ++x) ok[h][x] = none;
#pragma unroll
                for (int s = 0; s < NS; ++s) g[h][s] = s == 0 ? S::ident : 0.f;
                if constexpr (OP == OP_LN_FWD) {  // a member's count follows from its slice
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
                                __hip_atomic_load(p[h] + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
            lanes_merge<R, NS>(g[0], 64, merge);
            if (lane < R) {
#pragma unroll
                for (int s = 0; s < NS; ++s) lds.xb[lane][s] = g[0][s];
            }
        }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                st[i][s] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(lds.xb[i][s])));
    }
}

// ---------------------------------------------------------------- the loop
template <int OP, int DT, int V, int R, bool FULL, bool SPLIT>
__device__ __forceinline__ void stream_rows(const RowArgs &a, int c, int grp, StreamLds<OP, R> &lds) {
    constexpr int EPV = Io<DT>::EPV, B = Io<DT>::BYTES, NP = stream_params(OP), NCP = stream_ncp(OP);
    constexpr bool TWO = two_in(OP);
    typedef StreamStat<OP> S;
    const int tid = threadIdx.x, T = (int)blockDim.x;
    int parity = 0;
    const float invN = 1.f / (float)a.N;
    // the slice: first vector, vectors (the partial one counted), full ones
    const int64_t c0 = (int64_t)c * a.chunk;
    const int64_t left = a.N - c0;
    const int nval = (int)(left <= 0 ? 0 : left < a.chunk ? left : a.chunk);
    const int nvec = (nval + EPV - 1) / EPV, nfv = nval / EPV, tn = nval - nfv * EPV;
    const int jp = nfv / T;  // slots before it are full in every lane, those after it empty
    // byte offset of each slot in its row; past the end: the row's last vector
    const uint32_t rowlast = (uint32_t)(a.N * B) - 16u;
    // (a slice of full slots needs one offset, the slots are uniform steps)
    constexpr int VO = FULL ? 1 : V;
    uint32_t off[VO];
#pragma unroll
    for (int j = 0; j < VO; ++j) {
        const uint32_t o = (uint32_t)(c0 * B) + (uint32_t)(j * T + tid) * 16u;
        off[j] = FULL || o < rowlast ? o : rowlast;
    }
    auto step_of = [&](int j) -> uint32_t { return FULL ? (uint32_t)(j * T) * 16u : 0u; };
    auto vo = [](int j) -> int { return FULL ? 0 : j; };
    // lanes of slot jp: whole vector, the row's partial vector, or nothing
    const int vjp = jp * T + tid;
    const bool lane_full = vjp < nfv, lane_part = vjp == nfv && tn > 0;
    const int lo = lane_part ? EPV - tn : 0;  // first own element of the partial vector
    auto own = [&](int i) -> bool { return (lane_full || lane_part) && i >= lo; };

    float par[NP ? NP : 1][NP ? V * EPV : 1];
    if constexpr (NP > 0) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const char *src = (const char *)(p == 0 ? a.gamma : a.beta);
#pragma unroll
            for (int j = 0; j < V; ++j)
#pragma unroll
                for (int i = 0; i < EPV; i += 4) {
                    const f32x4 v = *(const f32x4_u *)(src + (size_t)(off[vo(j)] + step_of(j)) * (4 / B) + 4 * i);
                    par[p][j * EPV + i] = v.x; par[p][j * EPV + i + 1] = v.y;
                    par[p][j * EPV + i + 2] = v.z; par[p][j * EPV + i + 3] = v.w;
                }
        }
    }
    float cp[NCP ? NCP : 1][NCP ? V * EPV : 1];
    if constexpr (NCP > 0) {
#pragma unroll
        for (int p = 0; p < NCP; ++p)
#pragma unroll
            for (int i = 0; i < V * EPV; ++i) cp[p][i] = 0.f;
    }
    // elements of this wave (LayerNorm forward)
    float held = 0.f;
    if constexpr (OP == OP_LN_FWD) {
        if constexpr (FULL) {
            held = 64.f * V * EPV;
        } else {
            float h = 0.f;
#pragma unroll
            for (int j = 0; j < V; ++j)
                h += j < jp ? (float)EPV : j > jp ? 0.f : lane_full ? (float)EPV : lane_part ? (float)tn : 0.f;
            held = wave_sum(h);
        }
    }
    const float inv_held = held > 0.f ? 1.f / held : 0.f;
    // lanes that hold an element of slot 0, as a reciprocal of their number
    const bool lane0 = FULL || jp > 0 || lane_full || lane_part;
    float inv_l0 = 0x1p-6f;
    if constexpr (OP == OP_LN_FWD && !FULL) {
        const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane0));
        inv_l0 = n ? 1.f / (float)n : 0.f;
    }

    u32x4 x0[R][V], x1[TWO ? R : 1][TWO ? V : 1];
    u32x4 n0[R][V], n1[TWO ? R : 1][TWO ? V : 1];
    float kf[R], nkf[R];     // first element of each row (LayerNorm forward)
    float sm[R], sr[R], nsm[R], nsr[R];  // saved mean and rstd (norm backward)
    // Loads of the round at row0.  `live` == 0: there is no such round, every
    // lane reads the first vector of the last valid rows again (one line).
    auto issue = [&](int64_t row0, uint32_t live) {
        uint32_t lo[VO];  // opaque: SGPR base + VGPR offset addressing (resident.h)
#pragma unroll
        for (int j = 0; j < VO; ++j) {
            lo[j] = off[j] & live;
            asm volatile("" : "+v"(lo[j]));
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t row = row0 + i < a.M ? row0 + i : row0;
            const char *r0 = (const char *)a.in0 + row * a.ld0 * B;
            const char *r1 = TWO ? (const char *)a.in1 + row * a.ld1 * B : nullptr;
#pragma unroll
            for (int j = 0; j < V; ++j) n0[i][j] = vload_nt<false>(r0 + (step_of(j) & live), lo[vo(j)]);
            if constexpr (TWO) {
#pragma unroll
                for (int j = 0; j < V; ++j) n1[i][j] = vload_nt<false>(r1 + (step_of(j) & live), lo[vo(j)]);
            }
            if constexpr (OP == OP_LN_FWD) {
                if constexpr (DT == DT_F32) nkf[i] = *(const float *)r0;
                else nkf[i] = __uint_as_float((unsigned)*(const unsigned short *)r0 << 16);
            }
            if constexpr (NCP > 0) {
                if constexpr (OP == OP_LN_BWD) nsm[i] = a.mean_in[row];
                nsr[i] = a.rstd_in[row];
            }
        }
    };
    // elements of a slot that are not the lane's own become 0
    auto mask = [&](u32x4 &d, int j) {
        if constexpr (!FULL) {
            if (j < jp) return;
            if (j > jp) {
                d = u32x4{0u, 0u, 0u, 0u};
                return;
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                unsigned m = 0u;
                if constexpr (B == 4) m = own(w) ? 0xffffffffu : 0u;
                else m = (own(2 * w) ? 0xffffu : 0u) | (own(2 * w + 1) ? 0xffff0000u : 0u);
                d[w] &= m;
            }
        }
    };
    // Stores of a slot of a row's output.  They are unconditional instructions,
    // so that the next round's wait for its loads need not wait for them as
    // well (a store behind a branch may not have been issued, and the counter
    // is then waited down to zero): a lane without a whole vector addresses
    // past the buffer's end and an absent row's buffer is empty, which drops
    // the store.  Only the one partial vector is stored by elements.
    uint32_t so[VO];  // off, made opaque every round
    auto store = [&](int64_t row, bool live, int j, u32x4 v) {
        char *orow = (char *)a.out + row * a.ldo * B;
        // the slot's step goes into the buffer's base: a scalar offset in the
        // store would drop the wait state that 16-byte store data needs
        __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            orow + step_of(j), 0, live ? (int)((uint32_t)(a.N * B) - step_of(j)) : 0, 0x00020000);
        const bool full = FULL || j < jp || (j == jp && lane_full);
        __builtin_amdgcn_raw_buffer_store_b128(v, rs, full ? so[vo(j)] : 0x80000000u, 0,
                                                CREDIT_STORE_NT ? 2 : 0);
        if (!FULL && live && j == jp && lane_part) {
#pragma unroll
            for (int i = 1; i < EPV; ++i) {
                if (i < lo) continue;
                char *p = orow + off[vo(j)] + i * B;
                if constexpr (B == 4) *(unsigned *)p = v[i];
                else *(unsigned short *)p = (unsigned short)(v[i / 2] >> (16 * (i & 1)));
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
            if constexpr (OP == OP_LN_FWD) kf[i] = nkf[i];
            if constexpr (NCP > 0) { sm[i] = OP == OP_LN_BWD ? nsm[i] : 0.f; sr[i] = nsr[i]; }
        }
        const int64_t nrow = row0 + step;
        // The wave that polls the exchange may issue its loads after it: loads
        // return in order, and its polls would wait for them.  Only the longest
        // rounds leave those loads time to arrive (LayerNorm backward, 4 rows of 2
        // BF16 vectors, 2048 x 131072 k = 16: 343 -> 327 us; LayerNorm forward k = 8
        // 198 against 211, RMSNorm backward k = 16 313 against 338).
        constexpr bool LATE = SPLIT && OP == OP_LN_BWD && V == 2 && R == 4;
        const bool poller = LATE && T > 64 && __builtin_amdgcn_readfirstlane(tid >> 6) == 0;
        auto next = [&]() { issue(nrow < a.M ? nrow : row0, nrow < a.M ? 0xffffffffu : 0u); };
        if (!poller) next();
        __builtin_amdgcn_sched_barrier(0);
        const int nr = (int)(a.M - row0 < R ? a.M - row0 : R);
#pragma unroll
        for (int j = 0; j < VO; ++j) {
            so[j] = off[j];
            asm volatile("" : "+v"(so[j]));
        }
        const bool writer = c == 0 && tid == 0;
        // each pass decodes the packed rows again (resident.h)
        auto fresh = [&]() {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                opaque<V>(x0[i]);
                if constexpr (TWO) opaque<V>(x1[i]);
            }
        };
        if constexpr (OP == OP_RMS_FWD || OP == OP_LN_FWD) {
            float st[R][S::NS];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if constexpr (OP == OP_RMS_FWD) {
                    float s = 0.f;
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        mask(x0[i][j], j);
                        float q[EPV];
                        decode<DT>(x0[i][j], q, 1.f);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) s = fmaf(q[e], q[e], s);
                        keep_order(s);
                    }
                    st[i][0] = wave_sum(s);
                } else {
                    // moments about the mean of one own element per lane, then
                    // (count, mean about the row's first element, M2) of the
                    // wave.  A lane past the slice has no vote: all of them hold
                    // the row's last vector, and a large first element of it
                    // would draw the shift away from the mean (rows of 132
                    // elements with one 100 spreads out: error of rstd up to 300
                    // roundings, 3 without)
                    float q[EPV];
                    decode<DT>(x0[i][0], q, 1.f);
                    const float q0 = !FULL && jp == 0 && lane_part ? q[EPV - 1] : q[0];
                    const float ms = wave_sum(lane0 ? q0 * inv_l0 : 0.f);
                    float s1 = 0.f, s2 = 0.f;
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        if (!FULL && j > jp) continue;
                        decode<DT>(x0[i][j], q, 1.f);
                        if (FULL || j < jp) {
#pragma unroll
                            for (int e = 0; e < EPV; ++e) {
                                const float d = q[e] - ms;
                                s1 += d;
                                s2 = fmaf(d, d, s2);
                            }
                        } else {
#pragma unroll
                            for (int e = 0; e < EPV; ++e) {
                                const float d = own(e) ? q[e] - ms : 0.f;
                                s1 += d;
                                s2 = fmaf(d, d, s2);
                            }
                        }
                        keep_order(s1, s2);
                    }
                    s1 = wave_sum(s1);
                    s2 = wave_sum(s2);
                    const float m = s1 * inv_held;
                    st[i][0] = held;
                    st[i][1] = held > 0.f ? (ms - kf[i]) + m : 0.f;
                    // held at 0 from below, but not where it is NaN (a row with a
                    // NaN or an infinity): fmaxf would make that 0
                    const float m2 = s2 - s1 * m;
                    st[i][2] = held > 0.f && !(m2 < 0.f) ? m2 : 0.f;
                }
            }
            stream_reduce<OP, R, SPLIT>(st, a, row0, nr, c, lds, parity);
            fresh();
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const float mean = OP == OP_LN_FWD ? kf[i] + st[i][S::NS - 2 < 0 ? 0 : S::NS - 2] : 0.f;
                const float rstd = rsqrtf(st[i][S::NS - 1] * invN + a.eps);
                if (writer && i < nr) {
                    if (a.mean_out) a.mean_out[row0 + i] = mean;
                    if (a.rstd_out) a.rstd_out[row0 + i] = rstd;
                }
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    float q[EPV], y[EPV];
                    decode<DT>(x0[i][j], q, 1.f);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) {
                        if constexpr (OP == OP_LN_FWD)
                            y[e] = fmaf((q[e] - mean) * rstd, par[0][j * EPV + e], par[NP - 1][j * EPV + e]);
                        else
                            y[e] = q[e] * rstd * par[0][j * EPV + e];
                    }
                    store(row0 + i, i < nr, j, encode<DT>(y, 1.f));
                }
            }
        } else if constexpr (OP == OP_LN_BWD || OP == OP_RMS_BWD) {
            constexpr bool LN = OP == OP_LN_BWD;
            float st[R][S::NS];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                float sg = 0.f, sgx = 0.f;
                const float mean = sm[i], rstd = sr[i];
                // an absent row of the last round (a copy of the first, never
                // stored) adds nothing to the column sums: its dy is 0
                const bool live = i < nr;
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    if (!FULL && j > jp) continue;
                    mask(x0[i][j], j);
                    mask(x1[i][j], j);
                    if (i > 0)
#pragma unroll
                        for (int w = 0; w < 4; ++w) x1[i][j][w] = live ? x1[i][j][w] : 0u;
                    float x[EPV], dy[EPV];
                    decode<DT>(x0[i][j], x, 1.f);
                    decode<DT>(x1[i][j], dy, 1.f);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) {
                        const float xh = (x[e] - mean) * rstd;
                        const float g = dy[e] * par[0][j * EPV + e];
                        sgx = fmaf(g, xh, sgx);
                        cp[0][j * EPV + e] = fmaf(dy[e], xh, cp[0][j * EPV + e]);
                        if constexpr (LN) {
                            sg += g;
                            cp[NCP - 1][j * EPV + e] += dy[e];
                        }
                    }
                    // the column sums are added here, not sunk past the row's
                    // reduction with the decoded slot kept alive for them
#pragma unroll
                    for (int p = 0; p < NCP; ++p)
#pragma unroll
                        for (int e = 0; e < EPV; ++e) keep1(cp[p][j * EPV + e]);
                    keep_order(sg, sgx);
                }
                if constexpr (LN) {
                    st[i][0] = wave_sum(sg);
                    st[i][1] = wave_sum(sgx);
                } else {
                    st[i][0] = wave_sum(sgx);
                }
            }
            stream_reduce<OP, R, SPLIT>(st, a, row0, nr, c, lds, parity);
            if constexpr (LATE)
                if (poller) next();
            fresh();
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const float mean = sm[i], rstd = sr[i];
                const float c1 = LN ? st[i][0] * invN : 0.f, c2 = st[i][LN ? 1 : 0] * invN;
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    float x[EPV], dy[EPV], dx[EPV];
                    decode<DT>(x0[i][j], x, 1.f);
                    decode<DT>(x1[i][j], dy, 1.f);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) {
                        const float xh = (x[e] - mean) * rstd;
                        dx[e] = rstd * (dy[e] * par[0][j * EPV + e] - c1 - xh * c2);
                    }
                    store(row0 + i, i < nr, j, encode<DT>(dx, 1.f));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }

    if constexpr (NCP > 0) {
#pragma unroll
        for (int p = 0; p < NCP; ++p) {
            float *dst = a.colpart + ((int64_t)grp * NCP + p) * a.N;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if (!FULL && j > jp) continue;
                float *d = dst + (off[vo(j)] + step_of(j)) / B;
                if (FULL || j < jp || lane_full) {
#pragma unroll
                    for (int e = 0; e < EPV; e += 4) {
                        const f32x4 v = {cp[p][j * EPV + e], cp[p][j * EPV + e + 1], cp[p][j * EPV + e + 2],
                                         cp[p][j * EPV + e + 3]};
                        *(f32x4_u *)(d + e) = v;
                    }
                } else if (lane_part) {
#pragma unroll
                    for (int e = 1; e < EPV; ++e)
                        if (e >= lo) d[e] = cp[p][j * EPV + e];
                }
            }
        }
    }
}

// FULL: every slice holds exactly V vectors per thread (N = k V T vectors).
template <int OP, int DT, int V, int R, bool SPLIT, bool FULL>
__global__ __launch_bounds__(64 * stream_max_waves(OP, DT, V, R)) void k_stream(RowArgs a) {
    if (SPLIT && a.epoch == 0u && a.epoch_ptr)
        a.epoch = __hip_atomic_load(a.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __shared__ StreamLds<OP, R> lds;
    int c = 0, grp = blockIdx.x;
    if constexpr (SPLIT) member_of(a, blockIdx.x, c, grp);
    stream_rows<OP, DT, V, R, FULL, SPLIT>(a, c, grp, lds);
}

}  // namespace credit
