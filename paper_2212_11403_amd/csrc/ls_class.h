// Haplotype classes: within a block of B consecutive variants (B = 16, 32 or
// 64), donors that carry the same alleles at all of them form one class. The
// recursions treat the members of a class alike, so a sweep can carry one
// pair of values per class instead of one value per donor through the block
// (ls_csweep.h). ls_model_init builds the classes of every block beside the
// internal rows when that is predicted to pay (choose_classes).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ls_internal.h"

namespace lsk {

// Class words (64 classes each) and donor words per wave that the class
// sweeps are instantiated for, where the registers of both fit a wave at two
// waves per SIMD.
#define LS_MENU_CLASS(X) X(2) X(3) X(4) X(6) X(8) X(10) X(12) X(16)
#define LS_MENU_CSLOT_A(X) X(4) X(8) X(16) X(24) X(32) X(40)
#define LS_MENU_CSLOT_B(X) X(48) X(64) X(80)
#define LS_MENU_CSLOT_C(X) X(96) X(112)
#define LS_MENU_CSLOT_D(X) X(128) X(144)
#define LS_MENU_CSLOT_E(X) X(160)
constexpr int kClassMaxWords = 16;
__host__ __device__ constexpr bool csweep_exists(int nslot, int kw, int vgpr_per_slot) {
    return (nslot + 4 * kw) * vgpr_per_slot + (vgpr_per_slot == 2 ? 60 : 45) <= 256;
}
// Register need of a class sweep: the donor words, four values per class word
// and about 45 more; the kernels are compiled for the waves per SIMD it gives.
__host__ __device__ constexpr int csweep_waves_per_simd(int nslot, int ks, int vgpr_per_slot) {
    const int need = (nslot + 4 * ks) * vgpr_per_slot + (vgpr_per_slot == 2 ? 60 : 45);
    const int w = 512 / ((need + 7) / 8 * 8);
    return w > 8 ? 8 : (w < 1 ? 1 : w);
}
__host__ __device__ constexpr int csweep_max_waves(int nslot, int ks, int vgpr_per_slot) {
    const int w = 4 * csweep_waves_per_simd(nslot, ks, vgpr_per_slot);
    return w > 8 ? 8 : w;
}

constexpr int kClassMinB = 16;   // shortest block
constexpr int kClassMinN = 512;  // below, one wave holds few donors: no gain
constexpr int kClassMaxN = 64 * 8 * 160;  // above, no class sweep holds the donors in registers
constexpr int kClassMinL = 64;

// Most classes a block may have: at most a quarter of the donors (more
// gains nothing) and what the sweeps are instantiated for.
inline int32_t class_cap(int32_t N) {
    const int32_t k = N / 4 / 64 * 64;
    return k < 64 * kClassMaxWords ? k : 64 * kClassMaxWords;
}
inline bool class_section(int32_t N, int32_t L) {
    return N >= kClassMinN && N <= kClassMaxN && L >= kClassMinL;
}

// Byte offsets of the class section of the model workspace, from its start
// (256-byte aligned). Arrays over blocks are sized for the shortest block.
struct ClassLayout {
    size_t off_max;    // int32 [4]: largest class count of a block, per block length
    size_t off_lr;     // double [L]: sum of log(1 - rho_m) over m < l
    size_t off_g64;    // double [L+1]: jump factors (see class_tables_kernel)
    size_t off_g32;    // float [L+1]
    size_t off_r64;    // double [L]: mu / (1 - mu) per variant (vector mu)
    size_t off_keys;   // uint64 [nblk][cap]: alleles of a class, bit b = variant b of the block
    size_t off_cnt;    // float [nblk][cap]: members of a class
    size_t off_rows;   // uint64 [L][cap/64]: class alleles at a variant, 64 classes a word
    size_t off_ids;    // uint32 [nblk][64 ceil(N/128)]: classes of the donors (see class_build_kernel)
    size_t total;
};
inline ClassLayout class_layout(int32_t N, int32_t L) {
    ClassLayout c;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) / 256 * 256;
        return at;
    };
    const size_t cap = (size_t)class_cap(N), l = (size_t)L;
    const size_t nblk = (l + kClassMinB - 1) / kClassMinB;
    c.off_max = take(4 * sizeof(int32_t));
    c.off_lr = take(l * sizeof(double));
    c.off_g64 = take((l + 1) * sizeof(double));
    c.off_g32 = take((l + 1) * sizeof(float));
    c.off_r64 = take(l * sizeof(double));
    c.off_keys = take(nblk * cap * sizeof(uint64_t));
    c.off_cnt = take(nblk * cap * sizeof(float));
    c.off_rows = take(l * (cap / 64) * sizeof(uint64_t));
    c.off_ids = take(nblk * (size_t)((N + 127) / 128) * 64 * sizeof(uint32_t));
    c.total = off;
    return c;
}

// Largest class count of any block of 16, 32 and 64 variants into most[0..2]
// (atomic maxima; above `cap`: more than cap, for this length or a shorter
// one). `most` holds 0 before.
hipError_t launch_class_count(const uint64_t *Hr, int64_t hr_stride, int32_t N, int32_t L,
                              int32_t cap, int32_t *most, hipStream_t st);
// Classes of every block of length 2^lb, at most 64 kw each (kw words a row).
hipError_t launch_class_build(const uint64_t *Hr, int64_t hr_stride, int32_t N, int32_t L, int lb,
                              int kw, char *section, const ClassLayout &lay, hipStream_t st);
// The per-variant tables lr, g64, g32 and, with a vector mu, r64.
hipError_t launch_class_tables(const double *rho, const double *mu_vec, int32_t N, int32_t L,
                               char *section, const ClassLayout &lay, hipStream_t st);

// Class sweeps over the donor-word menu, one function per group of it.
#define LS_DECLARE_CSWEEP(G)                                                                  \
    hipError_t launch_csweep_##G(const SweepPtrs &p, const ClassPtrs &c, const SweepArgs &a, \
                                 hipStream_t st);
LS_DECLARE_CSWEEP(f32_a)
LS_DECLARE_CSWEEP(f32_b)
LS_DECLARE_CSWEEP(f32_c)
LS_DECLARE_CSWEEP(f32_d)
LS_DECLARE_CSWEEP(f32_e)
LS_DECLARE_CSWEEP(f64_a)
LS_DECLARE_CSWEEP(f64_b)
#undef LS_DECLARE_CSWEEP
inline hipError_t launch_csweep(int prec, const SweepPtrs &p, const ClassPtrs &c,
                                const SweepArgs &a, hipStream_t st) {
    if (prec == 0)
        return c.nslot <= 40 ? launch_csweep_f64_a(p, c, a, st) : launch_csweep_f64_b(p, c, a, st);
    return c.nslot <= 40    ? launch_csweep_f32_a(p, c, a, st)
           : c.nslot <= 80  ? launch_csweep_f32_b(p, c, a, st)
           : c.nslot <= 112 ? launch_csweep_f32_c(p, c, a, st)
           : c.nslot <= 144 ? launch_csweep_f32_d(p, c, a, st)
                            : launch_csweep_f32_e(p, c, a, st);
}

// Shape and checkpoints of the class gradient for this workspace into
// ga.cg_* (cg_nslot = 0: the plain adjoint).
void plan_grad_class(GradArgs &ga, int prec);

}  // namespace lsk
