// The class sweep: the recursions of ls_sweep.h carried per haplotype class
// instead of per donor inside a block of B variants (ls_class.h).
//
// Both directions run v <- theta^l (.) (v + g_l S 1), S = sum(v), on a vector
// in free units: dividing the update of ls_sweep.h by its factor c leaves the
// jump factor g_l = rho / ((1 - rho)(N - 1)) and no factor on v; the product
// of the (1 - rho) comes from a prefix table in FP64 and powers of two are
// taken out whenever S leaves a range, so no step divides. Inside a block
// every member j of class k has v_j = P_k v0_j + Q_k, with v0 the vector at
// the start of the block, and
//   P <- theta P,   Q <- theta (Q + g S),   S = sum_k (A_k P_k + n_k Q_k),
// where A_k is the sum of v0 over the class and n_k its size (without the
// recipient). Wave 0 steps P and Q of all classes (lane = class, KS words of
// 64). Every wave keeps NSLOT words of the donor vector in registers; at the
// ends of a block it adds its donors to the sums of their classes, and forms
// the new v0 from (P, Q) of their classes.
//
// What bounds it: wave 0 issues about 5 KS + 30 vector instructions per
// variant (two masked multiplies under one EXEC word, an add and two FMAs
// per class word, then one wave sum); a block boundary costs about 5 vector
// instructions and two LDS accesses (the class's pair, the atomic add to its
// sum) per donor word, and LDS bounds it. P and Q are one read of 8 or 16
// bytes: with two reads N = 10,000 took 113 ns per step and compute unit
// instead of 89 (B = 32, kw = 10), N = 20,000 153 instead of 137 (64, 12),
// N = 10,000 in FP64 230 instead of 213 (32, 10). No step has a barrier. Each wave adds into its own
// copy of the sums, in program order, and the copies are added in wave
// order, so the results do not depend on scheduling.
#pragma once

#include <type_traits>

#include "ls_class.h"
#include "ls_device.h"

namespace lsk {

// P and Q scaled by r on the lanes of m ^ fl: one EXEC word for both.
#define LS_PM(op, i)                                                                       \
    "s_xor_b64 exec, %[m" #i "], %[fl]\n\t" op " %[p" #i "], %[r], %[p" #i "]\n\t" op      \
    " %[q" #i "], %[r], %[q" #i "]\n\t"
#define LS_PM_ARGS1 [p0] "+v"(p[0]), [q0] "+v"(q[0])
#define LS_PM_ARGS2 LS_PM_ARGS1, [p1] "+v"(p[1]), [q1] "+v"(q[1])
#define LS_PM_ARGS4 LS_PM_ARGS2, [p2] "+v"(p[2]), [q2] "+v"(q[2]), [p3] "+v"(p[3]), [q3] "+v"(q[3])
#define LS_PM_ARGS8                                                                         \
    LS_PM_ARGS4, [p4] "+v"(p[4]), [q4] "+v"(q[4]), [p5] "+v"(p[5]), [q5] "+v"(q[5]),        \
        [p6] "+v"(p[6]), [q6] "+v"(q[6]), [p7] "+v"(p[7]), [q7] "+v"(q[7])
#define LS_PM_IN1 [m0] "s"(m[0])
#define LS_PM_IN2 LS_PM_IN1, [m1] "s"(m[1])
#define LS_PM_IN4 LS_PM_IN2, [m2] "s"(m[2]), [m3] "s"(m[3])
#define LS_PM_IN8 LS_PM_IN4, [m4] "s"(m[4]), [m5] "s"(m[5]), [m6] "s"(m[6]), [m7] "s"(m[7])
#define LS_PM1(op) LS_PM(op, 0)
#define LS_PM2(op) LS_PM1(op) LS_PM(op, 1)
#define LS_PM4(op) LS_PM2(op) LS_PM(op, 2) LS_PM(op, 3)
#define LS_PM8(op) LS_PM4(op) LS_PM(op, 4) LS_PM(op, 5) LS_PM(op, 6) LS_PM(op, 7)
// n values of P and of Q from p and q, their words from m (n = 1, 2, 4 or 8)
#define LS_PM_DEFINE(T, op, n)                                                               \
    __device__ __forceinline__ void pair_scale##n(T *p, T *q, const uint64_t *m, uint64_t fl, \
                                                  T r) {                                     \
        uint64_t sv;                                                                         \
        asm("s_mov_b64 %[sv], exec\n\t" LS_PM##n(op) "s_mov_b64 exec, %[sv]"                 \
            : LS_PM_ARGS##n, [sv] "=&s"(sv)                                                  \
            : LS_PM_IN##n, [fl] "s"(fl), [r] "v"(r)                                          \
            : "scc");                                                                        \
    }
LS_PM_DEFINE(float, "v_mul_f32", 1)
LS_PM_DEFINE(float, "v_mul_f32", 2)
LS_PM_DEFINE(float, "v_mul_f32", 4)
LS_PM_DEFINE(float, "v_mul_f32", 8)
LS_PM_DEFINE(double, "v_mul_f64", 1)
LS_PM_DEFINE(double, "v_mul_f64", 2)
LS_PM_DEFINE(double, "v_mul_f64", 4)
LS_PM_DEFINE(double, "v_mul_f64", 8)
#undef LS_PM_DEFINE
#undef LS_PM_ARGS1
#undef LS_PM_ARGS2
#undef LS_PM_ARGS4
#undef LS_PM_ARGS8
#undef LS_PM_IN1
#undef LS_PM_IN2
#undef LS_PM_IN4
#undef LS_PM_IN8
#undef LS_PM1
#undef LS_PM2
#undef LS_PM4
#undef LS_PM8
#undef LS_PM
template <int KS, class T>
__device__ __forceinline__ void pair_scale_all(T (&p)[KS], T (&q)[KS], const uint64_t (&m)[KS],
                                               uint64_t fl, T r) {
    constexpr int n8 = KS / 8 * 8, n4 = KS / 4 * 4, n2 = KS / 2 * 2;
#pragma unroll
    for (int s = 0; s < n8; s += 8) pair_scale8(p + s, q + s, m + s, fl, r);
    if constexpr (n4 > n8) pair_scale4(p + n8, q + n8, m + n8, fl, r);
    if constexpr (n2 > n4) pair_scale2(p + n4, q + n4, m + n4, fl, r);
    if constexpr (KS > n2) pair_scale1(p + n2, q + n2, m + n2, fl, r);
}

// Exponent e with |x| in [2^e, 2^(e+1)) and powers of two, on normal values,
// by integer arithmetic (a wave-uniform x stays on the scalar unit).
__device__ __forceinline__ int exponent_of(float x) {
    return ((__float_as_int(x) >> 23) & 0xff) - 127;
}
__device__ __forceinline__ int exponent_of(double x) {
    return ((__double2hiint(x) >> 20) & 0x7ff) - 1023;
}
__device__ __forceinline__ float pow2(float, int e) { return __int_as_float((e + 127) << 23); }
__device__ __forceinline__ double pow2(double, int e) {
    return __hiloint2double((e + 1023) << 20, 0);
}

// v <- p v + q in v's own register (left to itself the compiler keeps both
// the old and the new donor vector live at the end of a block and spills).
__device__ __forceinline__ void fma_in_place(float &v, float p, float q) {
    asm("v_fma_f32 %0, %1, %0, %2" : "+v"(v) : "v"(p), "v"(q));
}
__device__ __forceinline__ void fma_in_place(double &v, double p, double q) {
    asm("v_fma_f64 %0, %1, %0, %2" : "+v"(v) : "v"(p), "v"(q));
}

template <class PT, int NSLOT, int KS, int DIR, bool MUV>
__global__ void __launch_bounds__(64 * csweep_max_waves(NSLOT, KS, PT::vgpr_per_slot))
__attribute__((amdgpu_waves_per_eu(csweep_waves_per_simd(NSLOT, KS, PT::vgpr_per_slot))))
csweep_kernel(const uint32_t *__restrict__ ids, const uint64_t *__restrict__ keys,
              const float *__restrict__ cnt, const uint64_t *__restrict__ rows,
              const double *__restrict__ lr, const typename PT::T *__restrict__ gt,
              const typename PT::T *__restrict__ rt, const double *__restrict__ mu_vec,
              const double *__restrict__ lu_prefix, const double *__restrict__ rho,
              const int32_t *__restrict__ recipients, typename PT::T *__restrict__ state,
              double *__restrict__ log_scale, uint32_t *__restrict__ status,
              typename PT::T *__restrict__ snap, const int lb, const double unit,
              const SweepArgs a) {
#pragma clang fp contract(off)
    using T = typename PT::T;
    constexpr int CK = 64 * KS;
    constexpr int E = CK + 64;  // LDS entries of a class array: entry 0 is no class's
    extern __shared__ __align__(16) char lds[];
    struct alignas(2 * sizeof(T)) Pair {
        T p, q;
    };
    Pair *const lpq = reinterpret_cast<Pair *>(lds);  // P and Q of every class

    const int nwaves = uniform(blockDim.x >> 6);
    const int wave = uniform(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int r = a.r0 + blockIdx.x;
    const int N = a.N;
    const int i = recipients[r];
    if (i < 0 || i >= N) {
        if (threadIdx.x == 0) status[r] |= kFlagBadRecipient;
        return;
    }
    // class sums, [nwaves][E]: in FP64 for both precisions, as the LDS adds FP32
    // values one lane after another (193 cycles per instruction and compute
    // unit, FP64 29)
    double *const sums = reinterpret_cast<double *>(lpq + E);
    double *const own = sums + wave * E;
    const bool fresh = a.l0 < 0;
    const T v_fresh = DIR == 0 ? (T)0 : (T)1;
    const int B = 1 << lb;
    const int idw = ((N + 127) >> 7) * 64;  // id words of a block
    // S is kept in [2^-LIM, 2^LIM], so P <= 2 / A after a renormalisation: below
    // 2^91 in FP32, as no donor's share falls below 2^-90 (the model's check,
    // share_fall). The clamp is for the class of the recipient alone, which
    // has no mass and no members: its P and Q grow while S falls, and are held
    // finite, as they meet the factors A = 0 and n = 0
    constexpr int LIM = sizeof(T) == 4 ? 24 : 64;
    const T big = pow2((T)0, sizeof(T) == 4 ? 100 : 900);

    // ---- the donor vector: slot s holds donors 64 (wave NSLOT + s) + lane -------
    T v[NSLOT];
    const int self_word = i >> 6;
    const uint64_t self_bit = 1ull << (i & 63);
    // The ids of a block hold 4 (class + 1), two donor words per id word; an
    // id outside the block's array reads as 0: entry 0, which holds P = Q = 0
    // (so a lane without a donor keeps the value 0).
    // The id words come in groups of 16, whose loads are in flight together;
    // `each` takes eight slots at a time.
    auto for_ids = [&](int m, auto &&each) __attribute__((always_inline)) {
        const rsrc_t rs = make_rsrc(ids + (int64_t)m * idw, (uint32_t)idw * 4u);
        const int word0 = opaque(wave * NSLOT);
#pragma unroll
        for (int s0 = 0; s0 < NSLOT; s0 += 32) {
            constexpr int G = NSLOT < 32 ? NSLOT : 32;
            uint32_t w[G / 2];
#pragma unroll
            for (int k = 0; k < G / 2; ++k)
                if (s0 + 2 * k < NSLOT)
                    w[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4,
                                                                (word0 + s0 + 2 * k) * 128, 0);
            // the recipient takes entry 0: its value is and stays 0
            if ((unsigned)(self_word - word0 - s0) < (unsigned)G) {
                const uint32_t keep = self_word & 1 ? 0xffffu : 0xffff0000u;
#pragma unroll
                for (int k = 0; k < G / 2; ++k)
                    if (s0 + 2 * k < NSLOT) {
                        const bool hit = (self_word ^ (word0 + s0 + 2 * k)) < 2;
                        w[k] = lane_bit(hit ? self_bit : 0ull) ? w[k] & keep : w[k];
                    }
            }
#pragma unroll
            for (int h = 0; h < G; h += 8) {
                if (s0 + h >= NSLOT) break;
                int id4[8] = {};
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (s0 + h + 2 * k < NSLOT) {
                        id4[2 * k] = (int)(w[h / 2 + k] & 0xffffu);
                        id4[2 * k + 1] = (int)(w[h / 2 + k] >> 16);
                    }
                each(s0 + h, NSLOT - s0 - h < 8 ? NSLOT - s0 - h : 8, word0 + s0 + h, id4);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    auto entry = [&](auto *array, int id4) __attribute__((always_inline)) -> decltype(array) {
        constexpr int W = (int)sizeof(*array) / 4;
        return reinterpret_cast<decltype(array)>(reinterpret_cast<char *>(array) + id4 * W);
    };
    auto scatter = [&](int m) __attribute__((always_inline)) {
        for (int k = lane; k < E; k += 64) own[k] = 0.0;
        for_ids(m, [&](int s, int cnt8, int, const int (&id4)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < cnt8)
                    __hip_atomic_fetch_add(entry(own, id4[k]), (double)v[s + k], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
        });
    };
    // (P, Q) of the donors of eight slots
    auto pairs_of = [&](int cnt8, const int (&id4)[8], T (&p)[8], T (&q)[8])
                        __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k < cnt8) {
                const Pair x = *entry(lpq, id4[k]);
                p[k] = x.p;
                q[k] = x.q;
            }
    };
    auto expand = [&](int m) __attribute__((always_inline)) {
        for_ids(m, [&](int s, int cnt8, int word, const int (&id4)[8]) __attribute__((always_inline)) {
            T p[8], q[8];
            pairs_of(cnt8, id4, p, q);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < cnt8) fma_in_place(v[s + k], p[k], q[k]);
        });
    };
    auto out_row = [&](int m, T *dst) __attribute__((always_inline)) {
        const rsrc_t rs = make_rsrc(dst, (uint32_t)N * (uint32_t)sizeof(T));
        for_ids(m, [&](int s, int cnt8, int word, const int (&id4)[8]) __attribute__((always_inline)) {
            T p[8], q[8];
            pairs_of(cnt8, id4, p, q);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < cnt8)
                    buf_store(fma(p[k], v[s + k], q[k]), rs, lane * (int)sizeof(T),
                              (word + k) * 64 * (int)sizeof(T), kStreaming);
        });
    };
    if (fresh) {
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) v[s] = v_fresh;
    } else {
        const rsrc_t rs = make_rsrc(state + (int64_t)r * N, (uint32_t)N * (uint32_t)sizeof(T));
#pragma unroll
        for (int s = 0; s < NSLOT; ++s)
            v[s] = buf_load<T>(rs, lane * (int)sizeof(T), (wave * NSLOT + s) * 64 * (int)sizeof(T));
    }

    // ---- class values (wave 0) ------------------------------------------------
    T P[KS], Q[KS], A[KS], n[KS];
    T S = (T)1, Sprev = (T)1;
    const T r_fix = in_vgpr((T)a.th_mis);
    int expo = 0;             // powers of two taken out of v
    double s_load = 1.0;      // forward, resumed: sum of the table's vector
    uint64_t own_key = 0;     // the recipient's alleles in this block
    auto total = [&]() __attribute__((always_inline)) -> T {
        T a0 = P[0] * A[0], a1 = Q[0] * n[0];
#pragma unroll
        for (int s = 1; s < KS; ++s) {
            a0 = fma(P[s], A[s], a0);
            a1 = fma(Q[s], n[s], a1);
        }
        T x = a0 + a1;
        // a DPP instruction needs five wait states after a scalar write of
        // EXEC (the masked multiplies): the sum depends on all of them
        asm volatile("s_nop 4" : "+v"(x));
        return wave_sum(x);
    };
    // start of block m
    auto open_block = [&](int m, bool first) __attribute__((always_inline)) {
        const uint32_t idp = ids[(int64_t)m * idw + (i >> 7) * 64 + (i & 63)];
        const int ci = uniform((int)((i & 64 ? idp >> 16 : idp & 0xffffu) / 4u) - 1);
        own_key = keys[(int64_t)m * CK + ci];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = s * 64 + lane;
            n[s] = (T)cnt[(int64_t)m * CK + k] - (k == ci ? (T)1 : (T)0);
            A[s] = first && fresh ? n[s] * v_fresh : (T)0;
            P[s] = (T)1;
            Q[s] = (T)0;
        }
        if (!(first && fresh)) {
            double x[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) x[s] = sums[s * 64 + lane + 1];
            for (int w = 1; w < nwaves; ++w)
#pragma unroll
                for (int s = 0; s < KS; ++s) x[s] += sums[w * E + s * 64 + lane + 1];
#pragma unroll
            for (int s = 0; s < KS; ++s) A[s] = (T)x[s];
        }
        if (!(first && fresh && DIR == 0)) S = total();
        if (first && !fresh) s_load = (double)S;
    };
    auto write_pairs = [&](T f) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < KS; ++s) lpq[s * 64 + lane + 1] = Pair{P[s] * f, Q[s] * f};
    };
    // S back into its range, by a power of two
    auto renorm = [&]() __attribute__((always_inline)) {
        const int e = exponent_of(S);
        if (e < -LIM || e > LIM) {
            const T f = pow2((T)0, -e);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                P[s] = fmin(P[s] * f, big);
                Q[s] = fmin(Q[s] * f, big);
            }
            S *= f;
            Sprev *= f;
            expo += e;
        }
    };
    auto words_at = [&](int l, uint64_t (&w)[KS]) __attribute__((always_inline)) {
        const uint64_t *row = rows + (int64_t)l * KS;
#pragma unroll
        for (int s = 0; s < KS; ++s) w[s] = row[s];
    };
    // Q += g S: the donors that jump into variant l
    auto jump = [&](T g) __attribute__((always_inline)) {
        const T b = g * S;
#pragma unroll
        for (int s = 0; s < KS; ++s) Q[s] += b;
    };
    // theta^l and the new sum
    auto emit = [&](int l, const uint64_t (&w)[KS], T rr) __attribute__((always_inline)) {
        const uint64_t fl = uniform((int)((own_key >> (l & (B - 1))) & 1ull)) ? ~0ull : 0ull;
        const T rv = MUV ? in_vgpr(rr) : r_fix;
        pair_scale_all<KS>(P, Q, w, fl, rv);
        Sprev = S;
        S = total();
        renorm();
    };
    auto r_at = [&](int l) __attribute__((always_inline)) -> T {
        if constexpr (!MUV) return (T)a.th_mis;
        else if constexpr (sizeof(T) == 4) return rt[2 * l + 1];
        else return rt[l];
    };
    auto g_at = [&](int l) __attribute__((always_inline)) -> T { return gt[DIR == 0 ? l : l + 1]; };
    // `count` whole steps (jump and emission) from variant l on. The words
    // and factors of a variant are read while the one before is stepped; two
    // sets taken in turn, so that none is copied.
    struct Ahead {
        uint64_t w[KS];
        T g, r;
    };
    auto fetch = [&](Ahead &h, int l) __attribute__((always_inline)) {
        words_at(l, h.w);
        h.g = g_at(l);
        h.r = r_at(l);
    };
    auto run = [&](int l, int count) __attribute__((always_inline)) {
        if (count <= 0) return;
        constexpr int D = DIR == 0 ? 1 : -1;
        Ahead x, y;
        fetch(x, l);
        for (; count >= 2; count -= 2, l += 2 * D) {
            fetch(y, l + D);
            jump(x.g);
            emit(l, x.w, x.r);
            fetch(x, count > 2 ? l + 2 * D : l);
            jump(y.g);
            emit(l + D, y.w, y.r);
        }
        if (count > 0) {
            jump(x.g);
            emit(l, x.w, x.r);
        }
    };
    auto emit_at = [&](int l) __attribute__((always_inline)) {
        uint64_t w[KS];
        words_at(l, w);
        emit(l, w, r_at(l));
    };
    // factor that turns v at a stop into the vector of the tables
    auto out_factor = [&](int l) __attribute__((always_inline)) -> T {
        if constexpr (DIR == 0) {
            double u = unit;
            if constexpr (MUV) u = (1.0 - 2.0 * mu_vec[l]) + mu_vec[l];
            if (l > 0) u *= 1.0 - rho[l - 1];
            return (T)(u / (double)Sprev);
        } else {
            if (l == a.L - 1) return (T)1;
            return (T)((1.0 - rho[l]) * (double)(N - 1) / (double)S);
        }
    };
    // ---- march ------------------------------------------------------------
    // Wave 0 steps to the next event (a target, the end of the block or the
    // last variant); then all waves write the vector out or take it to the
    // next block.
    const int top = fresh ? a.L - 1 : a.l0;  // backward: the variant of the table
    const int lfirst = DIR == 0 ? (fresh ? 0 : a.l0 + 1) : top;
    int m = lfirst >> lb;
    int l = lfirst;  // next variant to step
    int kt = 0;
    bool held = true;  // backward: the jump into l is already in v (or there is none)
    if (threadIdx.x == 0) lpq[0] = Pair{(T)0, (T)0};
    if (!fresh) scatter(m);
    __syncthreads();
    if (wave == 0) open_block(m, true);
    for (;;) {
        bool block_end;
        bool tgt;
        if constexpr (DIR == 0) {
            const int bend = min(((m + 1) << lb) - 1, a.t);
            tgt = kt < a.nt && a.tgt_l[kt] <= bend;
            const int stop = tgt ? a.tgt_l[kt] : bend;
            block_end = !tgt && stop != a.t;
            if (wave == 0) run(l, stop - l + 1);
            l = stop + 1;
        } else {
            // a stop inside the block comes after the jump into its variant
            // and before its emission
            const int bend = max(m << lb, a.t);
            tgt = kt < a.nt && a.tgt_l[kt] >= bend;
            block_end = !tgt && bend != a.t;
            const int stop = tgt ? a.tgt_l[kt] : bend;
            const bool at_stop = !block_end && held && stop == l;
            if (wave == 0 && !at_stop) {
                if (held) emit_at(l);
                const int from = held ? l - 1 : l;
                run(from, from - stop + (block_end ? 1 : 0));
                if (!block_end) jump(g_at(stop));
            }
            held = !block_end;
            l = block_end ? stop - 1 : stop;
        }
        if (wave == 0) {
            T f;
            if (block_end) {  // the next v0 in units in which its sum is near 1
                const int e = exponent_of(S);
                f = pow2((T)0, -e);
                Sprev *= f;
                expo += e;
            } else {
                f = out_factor(DIR == 0 ? l - 1 : l);
            }
            write_pairs(f);
        }
        __syncthreads();
        if (block_end) {
            expand(m);
            m += DIR == 0 ? 1 : -1;
            scatter(m);
        } else {
            T *dst = tgt ? snap + (int64_t)a.tgt_out[kt] * a.snap_ts + (int64_t)r * a.snap_rs
                         : state + (int64_t)r * N;
            out_row(m, dst);
            if (!tgt) break;
            ++kt;
        }
        __syncthreads();
        if (wave == 0 && block_end) open_block(m, false);
    }
    // ---- epilogue: log scale and status -----------------------------------
    if (threadIdx.x == 0) {
        double ls = fresh ? 0.0 : log_scale[r];
        ls += (double)expo * 0.69314718055994530942 + log((double)S);
        if constexpr (DIR == 0) {
            if (!fresh) ls -= log(s_load);
            ls += lr[a.t] - lr[lfirst > 0 ? lfirst - 1 : 0];
            if constexpr (MUV) ls += lu_prefix[a.t + 1] - lu_prefix[lfirst];
            else ls += (double)(a.t - lfirst + 1) * log(unit);
        } else {
            // log G^t = log of the sum of y^{t+1} over N-1
            ls += lr[top] - lr[a.t + 1] - log((double)(N - 1));
            if constexpr (MUV) ls += lu_prefix[top + 1] - lu_prefix[a.t + 1];
            else ls += (double)(top - a.t) * log(unit);
        }
        log_scale[r] = ls;
        if (!isfinite(ls)) status[r] |= kFlagNonfinite;
    }
}

template <class PT, int NSLOT, int KS>
hipError_t launch_csweep_one(const SweepPtrs &p, const ClassPtrs &c, const SweepArgs &a,
                             hipStream_t st) {
    using T = typename PT::T;
    if (c.nwaves < 1 || c.nwaves > csweep_max_waves(NSLOT, KS, PT::vgpr_per_slot) ||
        (int64_t)c.nwaves * NSLOT * 64 < a.N || a.nblk < 1 || a.r0 < 0 || a.r0 + a.nblk > a.R)
        return hipErrorInvalidValue;
    // the kernel's limit is set to what its widest group takes, whatever this one
    // takes: it is one value of the process, and another thread may be about to
    // launch the same kernel with more waves
    auto bytes = [](int waves) { return (size_t)(64 * KS + 64) * (2 * sizeof(T) + waves * sizeof(double)); };
    const size_t lds = bytes(c.nwaves);
    auto go = [&](auto kern) {
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute(
                reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                (int)bytes(csweep_max_waves(NSLOT, KS, PT::vgpr_per_slot)));
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3(a.nblk), dim3(64 * c.nwaves), lds, st, c.ids, c.keys, c.cnt,
                           c.rows, c.lr, (const T *)c.g, (const T *)c.r, c.mu_vec, p.lu_prefix,
                           p.rho, p.recipients, (T *)p.state, p.log_scale, p.status, (T *)p.snap,
                           c.lb, c.unit, a);
        return hipGetLastError();
    };
    if (a.dir == 0)
        return p.emis ? go(&csweep_kernel<PT, NSLOT, KS, 0, true>)
                      : go(&csweep_kernel<PT, NSLOT, KS, 0, false>);
    return p.emis ? go(&csweep_kernel<PT, NSLOT, KS, 1, true>)
                  : go(&csweep_kernel<PT, NSLOT, KS, 1, false>);
}

// The class-word menu of one slot count (each instantiated in a file of its
// own group of slot counts, so that the build compiles them in parallel).
template <class PT, int NSLOT>
hipError_t launch_csweep_slots(const SweepPtrs &p, const ClassPtrs &c, const SweepArgs &a,
                               hipStream_t st) {
    switch (c.kw) {
#define LS_CASE(k)                                                    \
    case k:                                                           \
        if constexpr (csweep_exists(NSLOT, k, PT::vgpr_per_slot))     \
            return launch_csweep_one<PT, NSLOT, k>(p, c, a, st);      \
        return hipErrorInvalidValue;
        LS_MENU_CLASS(LS_CASE)
#undef LS_CASE
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace lsk
