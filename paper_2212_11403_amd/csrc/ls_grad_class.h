// The adjoint pass of the gradient carried per haplotype class (ls_class.h):
// the score of ls_grad_kernel.h, one workgroup per recipient, walking blocks
// of 2^lb variants from the last to the first.
//
// Inside a block the forward vector of donor j in class k is
//   alpha^l_j = P_k(l) a_j + Q_k(l),   a = the vector at the end of the block before,
// and the backward vector y^l = theta^l (.) beta^l is
//   y^l_j = P'_k(l) z_j + Q'_k(l),     z = y at the start of the block after,
// both in free units (the score is homogeneous in either). So with the class
// sums A = sum a, Y = sum z, X = sum a z and the class size n, the products
// over donors are sums over classes:
//   F1 = P X + Q Y,  F2 = P A + Q n   (P, Q at l),
//   d_l = sum_j alpha^l_j y^{l+1}_j = sum_k F1 P' + F2 Q'   (P', Q' at l+1),
//   Z_l = sum_j alpha^l_j beta^l_j  = sum_k F1 P' + F2 (Q' + g S'),
// and M_l is the part of Z_l in the classes that mismatch at l. The parts that
// mismatch and match are summed apart, so that M and 1 - M both keep their
// digits (a mutated site has M within 1e-3 of 1); and the FP32 rounding of the mismatch ratio,
// the same at every variant, is taken out of the odds M / (1 - M) in FP64.
// Error of d/dmu in FP32 at N = 2,000, L = 5,000, mu = 1e-4, relative to the
// summed magnitudes, over eight inputs: 5e-10; 1.7e-8 with M = Z_mismatch /
// (d + g S S') and the ratio as rounded, 1.2e-8 in the plain adjoint. Only z lives
// in registers; the a of a block are the checkpoints of the forward class
// sweep at every block end and are read once, for A and X.
//
// Wave 0 steps the classes. Forward through the block it keeps (P, Q) every
// eight variants in LDS and the jump g S of each variant in a lane of one
// register; backward, eight variants at a time, it forms their (P, Q) again
// in registers and steps P' and Q' through them. The scalars of a variant
// are kept in lane l mod 64, and the FP64 terms of a block are formed for all
// its variants at once.
//
// What bounds it: wave 0's vector instructions, per variant about 54 forward,
// 50 to form (P, Q) again and 135 backward at four class words, against some
// 180 of each of four waves and the recompute's stores of alpha in the plain
// adjoint. N = 2,000, L = 5,000, FP32, all recipients: 28.8 -> 6.2 ms per
// gradient step.
#pragma once

#include "ls_csweep.h"

namespace lsk {

struct GradClassArgs {
    int32_t N, L, R;
    int32_t lb;
    int32_t m_hi, m_lo;     // blocks of this launch, from m_hi down to m_lo
    int32_t vec_lo, vec_up; // checkpoint before block m_lo; before m > m_lo: vec_up + m - m_lo - 1
    double th_mis;          // emission of a mismatch (scalar mu), 1 for a match
    double inv_mu, inv_omu;
};

// Registers: the donor words, 8 (P, Q) pairs, P, Q, P', Q', A, X, Y, n and
// two words of mismatch bits per class word, and about 60 more.
__host__ __device__ constexpr int grad_class_regs(int nslot, int ks, int vgpr_per_slot) {
    return (nslot + 24 * ks) * vgpr_per_slot + 2 * ks + 60;
}
__host__ __device__ constexpr bool grad_class_exists(int nslot, int ks, int vgpr_per_slot) {
    return grad_class_regs(nslot, ks, vgpr_per_slot) <= 440;
}
__host__ __device__ constexpr int grad_class_waves_per_simd(int nslot, int ks, int vgpr_per_slot) {
    const int w = 512 / ((grad_class_regs(nslot, ks, vgpr_per_slot) + 7) / 8 * 8);
    return w > 8 ? 8 : (w < 1 ? 1 : w);
}
constexpr int kGradClassMaxWaves = 4;
// Most local memory a group may take; where a kernel needs its limit raised, it
// is raised to this, one value whatever the launch (see launch_csweep_one).
constexpr size_t kGradClassMaxLds = 128 * 1024;
// LDS bytes: class sums of every wave while donors are added up, then (P, Q)
// every eight variants, then (P', Q').
inline size_t grad_class_lds(int ks, int lb, int nwaves, size_t tsize) {
    const size_t e = 64 * (size_t)ks + 64;
    const size_t sums = 3 * e * sizeof(double) * (size_t)nwaves;
    const size_t kept = ((size_t)1 << lb) / 8 * 2 * 64 * (size_t)ks * tsize;
    const size_t pq = 2 * e * tsize;
    return sums > kept ? (sums > pq ? sums : pq) : (kept > pq ? kept : pq);
}

__device__ __forceinline__ float read_lane(float x, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ double read_lane(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Between two uses of the same local memory by one wave: its lanes' accesses on
// either side stay in order. The hardware keeps the order of a wave's own
// accesses; the compiler, to which the two uses are arrays of different types
// or different elements, need not.
__device__ __forceinline__ void reuse_lds() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");
    __builtin_amdgcn_wave_barrier();
}

template <class PT, int NSLOT, int KS, bool MUV>
__global__ void __launch_bounds__(64 * kGradClassMaxWaves)
__attribute__((amdgpu_waves_per_eu(grad_class_waves_per_simd(NSLOT, KS, PT::vgpr_per_slot))))
grad_class_kernel(const uint32_t *__restrict__ ids, const uint64_t *__restrict__ keys,
                  const float *__restrict__ cnt, const uint64_t *__restrict__ rows,
                  const typename PT::T *__restrict__ gt, const typename PT::T *__restrict__ rt,
                  const double *__restrict__ mu_vec, const double *__restrict__ rho,
                  const int32_t *__restrict__ recipients,
                  const typename PT::T *__restrict__ vecs, typename PT::T *__restrict__ ybuf,
                  double *__restrict__ grow, double *__restrict__ gmu, double *__restrict__ gmul,
                  const GradClassArgs a) {
#pragma clang fp contract(off)
    using T = typename PT::T;
    constexpr int CK = 64 * KS;
    constexpr int E = CK + 64;
    extern __shared__ __align__(16) char lds[];
    double *const sums = reinterpret_cast<double *>(lds);  // [nwaves][3][E]: A, X, Y
    T *const kept = reinterpret_cast<T *>(lds);            // [B / 8][2][CK]
    T *const lp = reinterpret_cast<T *>(lds);              // P', then Q'
    T *const lq = lp + E;

    const int nwaves = uniform(blockDim.x >> 6);
    const int wave = uniform(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x;
    const int N = a.N, L = a.L;
    const int i = recipients[r];
    if (i < 0 || i >= N) return;
    const int B = 1 << a.lb;
    const int idw = ((N + 127) >> 7) * 64;
    const bool top_launch = ((a.m_hi + 1) << a.lb) >= L;  // its first block holds variant L-1
    constexpr int LIM = sizeof(T) == 4 ? 24 : 64;
    const T big = pow2((T)0, sizeof(T) == 4 ? 100 : 900);
    const int self_word = i >> 6;
    const uint64_t self_bit = 1ull << (i & 63);
    const int word0 = wave * NSLOT;

    T z[NSLOT];
    {
        const rsrc_t rs = make_rsrc(ybuf + (int64_t)r * N, (uint32_t)N * (uint32_t)sizeof(T));
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) {
            const int j = (word0 + s) * 64 + lane;
            if (top_launch) z[s] = (j < N && j != i) ? (T)1 : (T)0;
            else z[s] = buf_load<T>(rs, lane * (int)sizeof(T), (word0 + s) * 64 * (int)sizeof(T));
        }
    }
    auto entry = [&](auto *array, int id4) __attribute__((always_inline)) -> decltype(array) {
        constexpr int W = (int)sizeof(*array) / 4;
        return reinterpret_cast<decltype(array)>(reinterpret_cast<char *>(array) + id4 * W);
    };
    // class ids of eight slots at a time (see csweep_kernel); the recipient
    // takes entry 0
    auto for_ids = [&](int m, auto &&each) __attribute__((always_inline)) {
        const rsrc_t rs = make_rsrc(ids + (int64_t)m * idw, (uint32_t)idw * 4u);
        const int w0 = opaque(word0);
#pragma unroll
        for (int s0 = 0; s0 < NSLOT; s0 += 8) {
            uint32_t w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (s0 + 2 * k < NSLOT)
                    w[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, (w0 + s0 + 2 * k) * 128, 0);
            int id4[8] = {};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (s0 + 2 * k < NSLOT) {
                    const bool hit = (self_word ^ (w0 + s0 + 2 * k)) < 2;
                    const uint32_t keep = self_word & 1 ? 0xffffu : 0xffff0000u;
                    const uint32_t x = lane_bit(hit ? self_bit : 0ull) ? w[k] & keep : w[k];
                    id4[2 * k] = (int)(x & 0xffffu);
                    id4[2 * k + 1] = (int)(x >> 16);
                }
            each(s0, NSLOT - s0 < 8 ? NSLOT - s0 : 8, w0 + s0, id4);
        }
    };
    double gm = 0.0;  // mu terms of the variants l = lane (mod 64)

    for (int m = a.m_hi; m >= a.m_lo; --m) {
        // ---- class sums of a, a z and z ------------------------------------------
        {
            double *const own = sums + wave * 3 * E;
            for (int k = lane; k < 3 * E; k += 64) own[k] = 0.0;
            const int vec = m == a.m_lo ? a.vec_lo : a.vec_up + m - a.m_lo - 1;
            const bool have = m > 0;  // block 0 starts from nothing
            const T *arow = vecs + ((int64_t)(have ? vec : 0) * a.R + r) * N;
            const rsrc_t rs = make_rsrc(arow, have ? (uint32_t)N * (uint32_t)sizeof(T) : 0u);
            for_ids(m, [&](int s, int cnt8, int word, const int (&id4)[8]) __attribute__((always_inline)) {
                T x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (k < cnt8)
                        x[k] = buf_load<T>(rs, lane * (int)sizeof(T), (word + k) * 64 * (int)sizeof(T));
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (k < cnt8) {
                        const double xa = (double)x[k], xz = (double)z[s + k];
                        double *e = entry(own, id4[k]);
                        __hip_atomic_fetch_add(e, xa, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_fetch_add(e + E, xa * xz, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_fetch_add(e + 2 * E, xz, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
            });
        }
        __syncthreads();
        if (wave == 0) {
            const int l0 = m << a.lb;
            const int nv = min(B, L - l0);
            // X and Y of a class are held times 2^-eY, eY the exponent of Y, and its P'
            // and Q' Y term accordingly with P' 2^eY: the same products, but a class
            // whose a and z are both small keeps its X in range (X alone has the square
            // of the smallest share)
            T A[KS], X[KS], Y[KS], n[KS];
            int eY[KS];
            uint64_t mis[KS];  // bit b: the class mismatches the recipient at variant l0 + b
            const uint32_t idp = ids[(int64_t)m * idw + (i >> 7) * 64 + (i & 63)];
            const int ci = uniform((int)((i & 64 ? idp >> 16 : idp & 0xffffu) / 4u) - 1);
            const uint64_t own_key = keys[(int64_t)m * CK + ci];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int k = s * 64 + lane;
                double xa = sums[k + 1], xx = sums[E + k + 1], xy = sums[2 * E + k + 1];
                for (int w = 1; w < nwaves; ++w) {
                    xa += sums[w * 3 * E + k + 1];
                    xx += sums[w * 3 * E + E + k + 1];
                    xy += sums[w * 3 * E + 2 * E + k + 1];
                }
                A[s] = (T)xa;
                eY[s] = xy > 0.0 ? exponent_of(xy) : 0;
                const double down = pow2(0.0, -eY[s]);
                X[s] = (T)(xx * down);
                Y[s] = (T)(xy * down);
                n[s] = (T)cnt[(int64_t)m * CK + k] - (k == ci ? (T)1 : (T)0);
                mis[s] = keys[(int64_t)m * CK + k] ^ own_key;
            }
            reuse_lds();  // the sums are read; `kept` takes their place
            auto r_at = [&](int l) __attribute__((always_inline)) -> T {
                if constexpr (!MUV) return (T)a.th_mis;
                else if constexpr (sizeof(T) == 4) return rt[2 * l + 1];
                else return rt[l];
            };
            // ---- forward: (P, Q) every eight variants, the jump of each -----------
            T vS = (T)0, vJ = (T)0, vF = (T)1;  // lane b: S, g S and the rescaling of variant l0 + b
            {
                T P[KS], Q[KS];
                T S;
                auto total = [&]() __attribute__((always_inline)) -> T {
                    T a0 = P[0] * A[0], a1 = Q[0] * n[0];
#pragma unroll
                    for (int s = 1; s < KS; ++s) {
                        a0 = fma(P[s], A[s], a0);
                        a1 = fma(Q[s], n[s], a1);
                    }
                    T x = a0 + a1;
                    asm volatile("s_nop 4" : "+v"(x));  // EXEC writes before DPP
                    return wave_sum(x);
                };
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    P[s] = (T)1;
                    Q[s] = (T)0;
                }
                S = m > 0 ? total() : (T)1;
                uint64_t wn[KS];
                auto words = [&](int l) __attribute__((always_inline)) {
#pragma unroll
                    for (int s = 0; s < KS; ++s) wn[s] = rows[(int64_t)l * KS + s];
                };
                words(l0);
                T gn = gt[l0], rn = r_at(l0);
                for (int b = 0; b < nv; ++b) {
                    if ((b & 7) == 0) {
                        T *to = kept + (b >> 3) * 2 * CK + lane;
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            to[s * 64] = P[s];
                            to[CK + s * 64] = Q[s];
                        }
                    }
                    uint64_t w[KS];
#pragma unroll
                    for (int s = 0; s < KS; ++s) w[s] = wn[s];
                    const T g = gn, rr = in_vgpr(rn);
                    const int ln = l0 + (b + 1 < nv ? b + 1 : b);
                    words(ln);
                    gn = gt[ln];
                    rn = r_at(ln);
                    const T jump = g * S;
#pragma unroll
                    for (int s = 0; s < KS; ++s) Q[s] += jump;
                    const uint64_t fl = uniform((int)((own_key >> b) & 1ull)) ? ~0ull : 0ull;
                    pair_scale_all<KS>(P, Q, w, fl, rr);
                    S = total();
                    T f = (T)1;
                    const int e = exponent_of(S);
                    if (e < -LIM || e > LIM) {
                        f = pow2((T)0, -e);
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            P[s] = fmin(P[s] * f, big);
                            Q[s] = fmin(Q[s] * f, big);
                        }
                        S *= f;
                    }
                    const bool here = lane_bit(1ull << b);
                    vS = here ? S : vS;
                    vJ = here ? jump : vJ;
                    vF = here ? f : vF;
                }
            }
            // ---- backward ---------------------------------------------------------
            T vd = (T)0, vM = (T)0, vY = (T)0, vZ = (T)0;  // lane b: d, Z of mismatches, S', Z of matches
            T Pb[KS], Qb[KS];
            T Sb;
            {
                T y = (T)0;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    Pb[s] = pow2((T)0, eY[s]);
                    Qb[s] = (T)0;
                    y += Y[s] * Pb[s];
                }
                Sb = wave_sum(y);
            }
            for (int b0 = (nv - 1) & ~7; b0 >= 0; b0 -= 8) {
                T HP[8][KS], HQ[8][KS];
                uint32_t bits[KS];
                {
                    T P[KS], Q[KS];
                    const T *from = kept + (b0 >> 3) * 2 * CK + lane;
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        P[s] = from[s * 64];
                        Q[s] = from[CK + s * 64];
                        bits[s] = (uint32_t)(mis[s] >> b0) & 0xffu;
                    }
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        if (b0 + t < nv) {
                            const T jump = read_lane(vJ, b0 + t), f = read_lane(vF, b0 + t);
                            const T rr = r_at(l0 + b0 + t);
#pragma unroll
                            for (int s = 0; s < KS; ++s) {
                                const T th = bits[s] & (1u << t) ? rr : (T)1;
                                P[s] *= th;
                                Q[s] = (Q[s] + jump) * th;
                            }
                            if (f != (T)1) {
#pragma unroll
                                for (int s = 0; s < KS; ++s) {
                                    P[s] = fmin(P[s] * f, big);
                                    Q[s] = fmin(Q[s] * f, big);
                                }
                            }
                        }
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            HP[t][s] = P[s];
                            HQ[t][s] = Q[s];
                        }
                    }
                }
#pragma unroll
                for (int t = 7; t >= 0; --t) {
                    if (b0 + t >= nv) continue;
                    const int l = l0 + b0 + t;
                    const T jump = gt[l + 1] * Sb;  // gt[L] = 0: beta^{L-1} = z
                    const T rr = r_at(l);
                    T d = (T)0, mn = (T)0, sy = (T)0, mt = (T)0;
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        const T F1 = fma(HP[t][s], X[s], HQ[t][s] * Y[s]);
                        const T F2 = fma(HP[t][s], A[s], HQ[t][s] * n[s]);
                        const T fp = F1 * Pb[s];
                        d += fma(F2, Qb[s], fp);
                        const T u = Qb[s] + jump;
                        const bool x = bits[s] & (1u << t);
                        const T zz = fma(F2, u, fp);
                        mn += x ? zz : (T)0;
                        mt += x ? (T)0 : zz;
                        const T th = x ? rr : (T)1;
                        Pb[s] *= th;
                        Qb[s] = u * th;
                        sy = fma(Pb[s], Y[s], fma(Qb[s], n[s], sy));
                    }
                    T q[4] = {d, mn, sy, mt}, w4[4];
                    wave_sum4(q, w4);
                    const bool here = lane_bit(1ull << (b0 + t));
                    vd = here ? w4[0] : vd;
                    vM = here ? w4[1] : vM;
                    vY = here ? Sb : vY;
                    vZ = here ? w4[3] : vZ;
                    Sb = w4[2];
                    const int e = exponent_of(Sb);
                    if (e < -LIM || e > LIM) {
                        const T f = pow2((T)0, -e);
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            Pb[s] = fmin(Pb[s] * f, big);
                            Qb[s] = fmin(Qb[s] * f, big);
                        }
                        Sb *= f;
                    }
                }
            }
            // ---- the terms of the block's variants, one per lane --------------------
            if (lane < nv) {
                const int l = l0 + lane;
                const double d = (double)vd, Sa = (double)vS, Sy = (double)vY;
                if (l < L - 1) {
                    const double rr = rho[l];
                    const double pss = Sa * Sy / (double)(N - 1);
                    grow[(int64_t)l * a.R + r] = (pss - d) / ((1.0 - rr) * d + rr * pss);
                }
                double zm = (double)vM;
                if constexpr (sizeof(T) == 4) {
                    double q;  // the mismatch ratio over its FP32 value
                    if constexpr (MUV) {
                        const double mu = mu_vec[l];
                        q = mu / (((1.0 - 2.0 * mu) + mu) * (double)rt[2 * l + 1]);
                    } else {
                        q = a.th_mis / (double)(float)a.th_mis;
                    }
                    zm *= q;
                }
                const double zt = zm + (double)vZ, M = zm / zt, M1 = (double)vZ / zt;
                if constexpr (MUV) {
                    const double mu = mu_vec[l];
                    gmul[(int64_t)l * a.R + r] = M / mu - M1 / ((1.0 - 2.0 * mu) + mu);
                } else {
                    gm += M * a.inv_mu - M1 * a.inv_omu;
                }
            }
            reuse_lds();  // `kept` is read; P' and Q' take its place
            // (P', Q') for the next z, in units in which its sum is near 1
            const T f = pow2((T)0, -exponent_of(Sb));
            if (lane == 0) lp[0] = lq[0] = (T)0;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                lp[s * 64 + lane + 1] = Pb[s] * f * pow2((T)0, -eY[s]);
                lq[s * 64 + lane + 1] = Qb[s] * f;
            }
        }
        __syncthreads();
        for_ids(m, [&](int s, int cnt8, int, const int (&id4)[8]) __attribute__((always_inline)) {
            T p[8], q[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < cnt8) {
                    p[k] = *entry(lp, id4[k]);
                    q[k] = *entry(lq, id4[k]);
                }
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < cnt8) fma_in_place(z[s + k], p[k], q[k]);
        });
        __syncthreads();
    }
    // hand y at the start of block m_lo to the launch below
    if (a.m_lo > 0) {
        const rsrc_t rs = make_rsrc(ybuf + (int64_t)r * N, (uint32_t)N * (uint32_t)sizeof(T));
#pragma unroll
        for (int s = 0; s < NSLOT; ++s)
            buf_store(z[s], rs, lane * (int)sizeof(T), (word0 + s) * 64 * (int)sizeof(T));
    }
    if (wave == 0) {
        const double g = wave_sum(gm);
        if (lane == 0) gmu[r] = (top_launch ? 0.0 : gmu[r]) + g;
    }
}

template <class PT, int NSLOT, int KS>
hipError_t launch_grad_class_one(const GradArgs &ga, const GradClassArgs &a, int nwaves,
                                 hipStream_t st) {
    using T = typename PT::T;
    const ClassPtrs &c = ga.cls;
    if (nwaves < 1 || nwaves > kGradClassMaxWaves || (int64_t)nwaves * NSLOT * 64 < a.N)
        return hipErrorInvalidValue;
    const size_t lds = grad_class_lds(KS, a.lb, nwaves, sizeof(T));
    if (lds > kGradClassMaxLds) return hipErrorInvalidValue;
    char *ws = ga.ws;
    const GradLayout &Ly = ga.lay;
    auto go = [&](auto kern) {
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)kGradClassMaxLds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3(a.R), dim3(64 * nwaves), lds, st, c.ids, c.keys, c.cnt, c.rows,
                           (const T *)c.g, (const T *)c.r, c.mu_vec, ga.rho, ga.recipients,
                           (const T *)(ws + Ly.off_ckpt), (T *)(ws + Ly.off_ybuf),
                           (double *)(ws + Ly.off_grow), (double *)(ws + Ly.off_gmu),
                           (double *)(ws + Ly.off_gmul), a);
        return hipGetLastError();
    };
    return ga.emis ? go(&grad_class_kernel<PT, NSLOT, KS, true>)
                   : go(&grad_class_kernel<PT, NSLOT, KS, false>);
}

// Donor words per wave of the class gradient; the class words are the class
// sweep's (LS_MENU_CLASS).
#define LS_MENU_GCLASS(X) X(8) X(16) X(24) X(32) X(40) X(48) X(64)

template <class PT>
hipError_t launch_grad_class_menu(const GradArgs &ga, const GradClassArgs &a, int nslot, int nwaves,
                                  hipStream_t st) {
#define LS_CASE2(n, k)                                                              \
    if constexpr (grad_class_exists(n, k, PT::vgpr_per_slot)) {                     \
        if (nslot == n && ga.cls.kw == k) return launch_grad_class_one<PT, n, k>(ga, a, nwaves, st); \
    }
#define LS_CASE(n) LS_CASE2(n, 2) LS_CASE2(n, 3) LS_CASE2(n, 4) LS_CASE2(n, 6) LS_CASE2(n, 8)
    LS_MENU_GCLASS(LS_CASE)
#undef LS_CASE
#undef LS_CASE2
    return hipErrorInvalidValue;
}

}  // namespace lsk
