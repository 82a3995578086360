// Builds the haplotype classes of a model (see ls_class.h).
#include <math.h>

#include "ls_class.h"
#include "ls_device.h"

namespace lsk {

namespace {

constexpr uint64_t kEmpty = ~0ull;

__device__ __forceinline__ uint32_t hash_key(uint64_t z) {
    z ^= z >> 31;
    z *= 0x9e3779b97f4a7c15ull;
    z ^= z >> 29;
    z *= 0xbf58476d1ce4e5b9ull;
    return (uint32_t)(z >> 32);
}

// Alleles of donor word * 64 + lane at variants l0 .. l0 + n - 1, variant
// l0 + b in bit b. `word` is wave-uniform: the rows are scalar loads, eight in
// flight (one at a time, a wave waits a memory latency per variant), and each
// is a lane mask as it stands, so a bit takes two instructions. Model set-up at
// N = 50,000, L = 2,000: 972 us, 1,529 with one load at a time.
__device__ __forceinline__ uint64_t donor_key(const uint64_t *__restrict__ Hr, int64_t stride,
                                              int NF, int word, int l0, int n) {
    const uint64_t *p = Hr + (int64_t)l0 * stride + (word < NF ? word : 2 * NF);
    uint64_t key = 0;
    for (int b = 0; b < n; b += 8) {
        uint64_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[(int64_t)min(b + u, n - 1) * stride];
        uint32_t bits = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) bits |= lane_bit(x[u]) ? 1u << u : 0u;
        if (n - b < 8) bits &= (1u << (n - b)) - 1u;
        key |= (uint64_t)bits << b;
    }
    return key;
}

// Hash slots: above cap + 1024 (each of the 1,024 threads may claim one more
// slot before it sees that the count has passed cap), so a probe always ends.
int hash_slots(int32_t cap) {
    int hs = 2048;
    while (hs < 2 * cap || hs < cap + 1088) hs *= 2;
    return hs;
}

// Slot of `key`, claimed if it is new; -1 once more than `cap` are claimed.
// The key that equals the empty mark has the extra slot HS.
__device__ __forceinline__ int find_slot(uint64_t key, unsigned long long *tab, int HS, int cap,
                                         int *count, int *extra) {
    if (key == kEmpty) {
        if (atomicExch(extra, 1) == 0) atomicAdd(count, 1);
        return HS;
    }
    int s = (int)(hash_key(key) & (uint32_t)(HS - 1));
    for (int probe = 0; probe < HS; ++probe) {
        unsigned long long old = tab[s];
        if (old == key) return s;
        if (old == kEmpty) {
            if (*(volatile int *)count > cap) return -1;
            old = atomicCAS(&tab[s], (unsigned long long)kEmpty, (unsigned long long)key);
            if (old == kEmpty) {
                atomicAdd(count, 1);
                return s;
            }
            if (old == key) return s;
        }
        s = (s + 1) & (HS - 1);
    }
    return -1;
}

}  // namespace

// One workgroup per block of variants, blocks of 16 first, then those of 32 and
// 64, in one launch (three launches left most of the card idle on short
// models). A block has at least the classes of its parts, so once a block has
// too many, blocks of that length and longer ones are not counted any more.
__global__ void __launch_bounds__(1024)
class_count_kernel(const uint64_t *__restrict__ Hr, int64_t stride, int32_t N, int32_t L, int HS,
                   int cap, int32_t *most) {
    extern __shared__ unsigned long long tab[];
    __shared__ int count, extra, skip;
    int blk = blockIdx.x, len = 0;  // length 16 << len
    for (; len < 2; ++len) {
        const int blocks = (L + (16 << len) - 1) >> (4 + len);
        if (blk < blocks) break;
        blk -= blocks;
    }
    const int l0 = blk << (4 + len);
    const int n = min(16 << len, L - l0);
    const int NF = N >> 6;
    for (int k = threadIdx.x; k < HS; k += 1024) tab[k] = kEmpty;
    if (threadIdx.x == 0) {  // one thread asks, so that all of them agree
        count = extra = skip = 0;
        for (int k = 0; k <= len; ++k)
            if (__hip_atomic_load(&most[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > cap) skip = 1;
        if (skip) atomicMax(&most[len], cap + 1);
    }
    __syncthreads();
    if (skip) return;
    const int lane = threadIdx.x & 63;
    for (int word = uniform(threadIdx.x >> 6); word * 64 < N; word += 16) {
        if (*(volatile int *)&count > cap) break;
        const uint64_t key = donor_key(Hr, stride, NF, word, l0, n);
        if (word * 64 + lane < N) find_slot(key, tab, HS, cap, &count, &extra);
    }
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(&most[len], count);
}

// Numbers the classes of a block by their first member (so the numbering
// does not depend on scheduling) and writes their alleles, sizes and rows,
// and every donor's class as 4 (class + 1), 0 for no donor (the byte offset
// of its entry in a class array). The caller has counted at most 64 kw classes.
__global__ void __launch_bounds__(1024)
class_build_kernel(const uint64_t *__restrict__ Hr, int64_t stride, int32_t N, int32_t L, int lb,
                   int HS, int kw, uint64_t *__restrict__ keys, float *__restrict__ cnt,
                   uint64_t *__restrict__ rows, uint16_t *__restrict__ ids) {
    extern __shared__ unsigned long long tab[];
    int *first = reinterpret_cast<int *>(tab + HS + 1);  // first member, then -1 - class
    int *members = first + HS + 1;
    __shared__ int count, extra, base, wcount[16];
    const int m = blockIdx.x;
    const int l0 = m << lb;
    const int n = min(1 << lb, L - l0);
    const int NF = N >> 6;
    const int cap = 64 * kw;
    for (int k = threadIdx.x; k <= HS; k += 1024) {
        tab[k] = kEmpty;
        first[k] = 0x7fffffff;
        members[k] = 0;
    }
    if (threadIdx.x == 0) count = extra = base = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    uint16_t *mine = ids + (int64_t)m * ((N + 127) / 128) * 128;
    // half-word of donor j: id word (j / 128) 64 + j % 64, half (j / 64) % 2
    auto at = [](int j) { return ((j >> 7) * 64 + (j & 63)) * 2 + ((j >> 6) & 1); };
    for (int word = wave; word * 64 < N; word += 16) {
        const int j = word * 64 + lane;
        const uint64_t key = donor_key(Hr, stride, NF, word, l0, n);
        if (j < N) {
            const int s = find_slot(key, tab, HS, cap, &count, &extra);
            if (s >= 0) {
                atomicMin(&first[s], j);
                atomicAdd(&members[s], 1);
            }
            mine[at(j)] = (uint16_t)(s < 0 ? 0 : s);
        }
    }
    __syncthreads();
    // classes in the order of their first members
    for (int j0 = 0; j0 < N; j0 += 1024) {
        const int j = j0 + threadIdx.x;
        const int s = j < N ? (int)mine[at(j)] : 0;
        const bool lead = j < N && first[s] == j;
        const uint64_t b = __ballot(lead);
        if (lane == 0) wcount[wave] = __popcll(b);
        __syncthreads();
        int before = base, total = base;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) before += wcount[w];
            total += wcount[w];
        }
        const int k = before + __popcll(b & ((1ull << lane) - 1ull));
        if (lead && k < cap) {
            keys[(int64_t)m * cap + k] = tab[s];
            cnt[(int64_t)m * cap + k] = (float)members[s];
            first[s] = -1 - k;
        }
        __syncthreads();
        if (threadIdx.x == 0) base = total;
        __syncthreads();
    }
    const int K = min(base, cap);
    for (int k = K + threadIdx.x; k < cap; k += 1024) {
        keys[(int64_t)m * cap + k] = 0;
        cnt[(int64_t)m * cap + k] = 0.0f;
    }
    for (int j = threadIdx.x; j < (N + 127) / 128 * 128; j += 1024) {
        const int f = j < N ? first[mine[at(j)]] : 0;
        mine[at(j)] = (uint16_t)(f < 0 ? -4 * f : 0);
    }
    __syncthreads();
    // the rows: lane b collects the word of variant b
    for (int q = wave; q < kw; q += 16) {
        const uint64_t key = keys[(int64_t)m * cap + q * 64 + lane];
        uint64_t word = 0;
        for (int b = 0; b < n; ++b) {
            const uint64_t w = __ballot((key >> b) & 1ull);
            word = lane == b ? w : word;
        }
        if (lane < n) rows[(int64_t)(l0 + lane) * kw + q] = word;
    }
}

hipError_t launch_class_count(const uint64_t *Hr, int64_t hr_stride, int32_t N, int32_t L,
                              int32_t cap, int32_t *most, hipStream_t st) {
    const int HS = hash_slots(cap);
    int blocks = 0;
    for (int lb = 4; lb <= 6; ++lb) blocks += (L + (1 << lb) - 1) >> lb;
    hipLaunchKernelGGL(class_count_kernel, dim3(blocks), dim3(1024), HS * sizeof(uint64_t), st, Hr,
                       hr_stride, N, L, HS, cap, most);
    return hipGetLastError();
}

hipError_t launch_class_build(const uint64_t *Hr, int64_t hr_stride, int32_t N, int32_t L, int lb,
                              int kw, char *section, const ClassLayout &lay, hipStream_t st) {
    const int HS = hash_slots(64 * kw);
    const int blocks = (L + (1 << lb) - 1) >> lb;
    const size_t lds = (size_t)(HS + 1) * (sizeof(uint64_t) + 2 * sizeof(int));
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&class_build_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(class_build_kernel, dim3(blocks), dim3(1024), lds, st, Hr, hr_stride, N, L,
                       lb, HS, kw, reinterpret_cast<uint64_t *>(section + lay.off_keys),
                       reinterpret_cast<float *>(section + lay.off_cnt),
                       reinterpret_cast<uint64_t *>(section + lay.off_rows),
                       reinterpret_cast<uint16_t *>(section + lay.off_ids));
    return hipGetLastError();
}

// g[0] = 1/(N-1), g[k] = rho_{k-1} / ((1 - rho_{k-1})(N-1)) for 0 < k < L,
// g[L] = 0: the jump into variant l adds g[l] S (forward) or g[l+1] S
// (backward) to every donor, in units in which a donor that does not jump
// keeps its value; lr[l] = sum of log(1 - rho_m), m < l, carries the rest.
// One workgroup: each thread sums a run of L/1024 variants, then the run
// totals are added in order.
__global__ void __launch_bounds__(1024)
class_tables_kernel(const double *__restrict__ rho, const double *__restrict__ mu_vec, int32_t N,
                    int32_t L, double *__restrict__ lr, double *__restrict__ g64,
                    float *__restrict__ g32, double *__restrict__ r64) {
    __shared__ double tot[1024];
    const int run = (L - 1 + 1023) / 1024;
    const int a = min(L - 1, (int)threadIdx.x * run), b = min(L - 1, a + run);
    const double n1 = (double)(N - 1);
    double s = 0.0;
    for (int l = a; l < b; ++l) s += log1p(-rho[l]);
    tot[threadIdx.x] = s;
    __syncthreads();
    for (int h = 1; h < 1024; h *= 2) {
        const double x = (int)threadIdx.x >= h ? tot[threadIdx.x - h] : 0.0;
        __syncthreads();
        tot[threadIdx.x] += x;
        __syncthreads();
    }
    s = threadIdx.x > 0 ? tot[threadIdx.x - 1] : 0.0;
    if (threadIdx.x == 0) {
        lr[0] = 0.0;
        g64[0] = 1.0 / n1;
        g32[0] = (float)(1.0 / n1);
        g64[L] = 0.0;
        g32[L] = 0.0f;
    }
    for (int l = a; l < b; ++l) {
        const double rr = rho[l];
        s += log1p(-rr);
        lr[l + 1] = s;
        const double g = rr / ((1.0 - rr) * n1);
        g64[l + 1] = g;
        g32[l + 1] = (float)g;
    }
    if (mu_vec)
        for (int l = threadIdx.x; l < L; l += 1024) {
            const double mu = mu_vec[l];
            r64[l] = mu / ((1.0 - 2.0 * mu) + mu);
        }
}

hipError_t launch_class_tables(const double *rho, const double *mu_vec, int32_t N, int32_t L,
                               char *section, const ClassLayout &lay, hipStream_t st) {
    hipLaunchKernelGGL(class_tables_kernel, dim3(1), dim3(1024), 0, st, rho, mu_vec, N, L,
                       reinterpret_cast<double *>(section + lay.off_lr),
                       reinterpret_cast<double *>(section + lay.off_g64),
                       reinterpret_cast<float *>(section + lay.off_g32),
                       reinterpret_cast<double *>(section + lay.off_r64));
    return hipGetLastError();
}

}  // namespace lsk
