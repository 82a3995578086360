// Consumers of the distance matrix: average pairwise linkage (the paper
// clusters a distance matrix with Sokal and Michener's method, section 6)
// and the standardisation of a recipient's half-distance row with the
// zero-deviation rule of section 2.2.
//
// Average linkage is a sequence of N-1 dependent merges, each cheap (a few
// passes over rows of N entries), so one workgroup runs all merges of one
// matrix and T matrices run side by side. The first nearest-neighbour pass
// reads every entry once and runs as its own kernel over all rows of all
// matrices, at full memory bandwidth.
//
// State per occupied slot k: nn[k], the occupied slot nearest to k (ties: the
// smallest slot), and nd[k], its distance. A merge takes the slot pair at the
// smallest distance (ties: the smallest slot pair; a NaN distance after every
// number), keeps the merged cluster in the smaller slot a, empties b, and
// updates row a and column a with d = (|A| d_a + |B| d_b) / (|A| + |B|)
// (each operation rounded in that order). Rows whose nearest slot was a or b
// are rescanned; every other row only compares its new distance to a.
//
// The pair at the smallest distance is (i, nn[i]) for the first slot i, in
// slot order, at the smallest nd: its nearest slot is then the smallest one at
// that distance, and were it below i, it would itself be at that distance and
// come before i. So a merge looks for the first smallest nd only.
//
// What bounds it: the chain of one merge, a handful of barriers and a round
// trip to memory (rows a and b, with the first four rescanned rows). Distances are
// compared as integers that order like them, so a wave finds a minimum with
// one DPP instruction per step; rows are rescanned four at a time by the whole
// workgroup, so their loads are in flight together; the barriers inside a
// merge wait for local memory only, and the one before the next merge also
// for the stores to D. Six FP32 matrices of N = 3,000: 20.7 ms, 6.9 us per
// merge (22.0 with the rescanned rows read after the update; 74.9 with pairs compared through shuffles, full barriers and one
// rescanned row after another).
#include <math.h>

#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "ls_cluster.h"
#include "ls_device.h"

namespace lsk {

namespace {

// (d1, p1) before (d2, p2): by distance, NaN after every number, then by slot.
template <class T>
__device__ __forceinline__ bool before(T d1, int p1, T d2, int p2) {
    const bool n1 = isnan(d1), n2 = isnan(d2);
    if (n1 != n2) return n2;
    if (!n1 && d1 != d2) return d1 < d2;
    return p1 < p2;
}

// Unsigned keys in the order of the distances: equal keys for equal distances
// (the two zeros included), every NaN after infinity, kNone after all.
__device__ __forceinline__ uint32_t order_key(float d) {
    if (isnan(d)) return 0xfffffffeu;
    const uint32_t u = __float_as_uint(d + 0.0f);
    return u & 0x80000000u ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ uint64_t order_key(double d) {
    if (isnan(d)) return ~0ull - 1ull;
    const uint64_t u = (uint64_t)__double_as_longlong(d + 0.0);
    return u >> 63 ? ~u : u | (1ull << 63);
}

template <int CTRL, int ROWMASK = 0xF>
__device__ __forceinline__ uint32_t dpp_min_u32(uint32_t x) {
    const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROWMASK, 0xF, false);
    return x < y ? x : y;
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    x = dpp_min_u32<0xB1>(x);         // quad_perm [1,0,3,2]
    x = dpp_min_u32<0x4E>(x);         // quad_perm [2,3,0,1]
    x = dpp_min_u32<0x124>(x);        // row_ror:4
    x = dpp_min_u32<0x128>(x);        // row_ror:8
    x = dpp_min_u32<0x142, 0xA>(x);   // row_bcast:15 into rows 1, 3
    x = dpp_min_u32<0x143, 0xC>(x);   // row_bcast:31 into rows 2, 3
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ uint64_t wave_min(uint64_t x) {
    const uint32_t hi = wave_min((uint32_t)(x >> 32));
    const uint32_t lo = wave_min((uint32_t)(x >> 32) == hi ? (uint32_t)x : ~0u);
    return (uint64_t)hi << 32 | lo;
}

// A candidate for the nearest slot: its key and slot (none: all ones).
template <class T>
struct Best {
    using K = decltype(order_key((T)0));
    K key = (K)~(K)0;
    uint32_t slot = ~0u;
    // a later candidate of the same thread, in slot order
    __device__ __forceinline__ void take(K k, uint32_t i) {
        if (k < key) {
            key = k;
            slot = i;
        }
    }
};
// The first candidate of a wave; `mine`: this lane holds it.
template <class T>
__device__ __forceinline__ Best<T> wave_best(Best<T> c, bool &mine) {
    Best<T> r;
    r.key = wave_min(c.key);
    r.slot = wave_min(c.key == r.key ? c.slot : ~0u);
    mine = c.key == r.key && c.slot == r.slot && r.slot != ~0u;
    return r;
}

// The best of one wave as the workgroup's reductions keep it.
template <class T>
struct WaveBest {
    typename Best<T>::K key;
    uint32_t slot;
    T d;
};

// Barrier of the workgroup for its local memory: global stores may still be
// on their way.
__device__ __forceinline__ void local_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace

// One wave per row: nn[k] and nd[k] of every row of every matrix.
template <class T>
__global__ void __launch_bounds__(256)
linkage_init_kernel(const T *__restrict__ D, int32_t N, int32_t T_, size_t ws_stride, char *ws) {
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= (int64_t)N * T_) return;
    const int t = (int)(row / N), i = (int)(row - (int64_t)t * N);
    char *w = ws + (size_t)t * ws_stride;
    int32_t *nn = reinterpret_cast<int32_t *>(w);
    T *nd = reinterpret_cast<T *>(w + 256 * (((size_t)N * 4 + 255) / 256));
    const T *r = D + ((int64_t)t * N + i) * N;
    Best<T> c;
    T d = (T)0;
#pragma unroll 4
    for (int k = threadIdx.x & 63; k < N; k += 64) {
        const T x = r[k];
        const auto key = order_key(x);
        if (k != i && key < c.key) {
            c.key = key;
            c.slot = (uint32_t)k;
            d = x;
        }
    }
    bool mine;
    wave_best(c, mine);
    if (mine) {
        nn[i] = (int32_t)c.slot;
        nd[i] = d;
    }
}

// Bytes of local memory the merge kernel keeps nn, nd and the rescan list of
// one matrix in (cluster sizes and ids stay in the workspace).
__host__ __device__ constexpr size_t linkage_lds_bytes(int32_t N, size_t tsize) {
    return 16 * (((size_t)N * tsize + 15) / 16) + 2 * (16 * (((size_t)N * 2 + 15) / 16));
}
constexpr int kLinkageLdsMaxN = 65535;  // slots are 16-bit there

// All N-1 merges of matrix blockIdx.x, then its leaf order. With SMEM nn
// (a slot's nearest slot; all ones: an empty slot), nd (its distance) and the
// rescan list live in local memory (linkage_lds_bytes), copied from the
// workspace the first pass filled, with 16-bit slots; else they stay in the
// workspace with 32-bit slots, and every barrier also waits for it.
template <class T, bool SMEM>
__global__ void __launch_bounds__(1024)
linkage_kernel(T *__restrict__ D, int32_t N, size_t ws_stride, char *ws, double *__restrict__ Z,
               int32_t *__restrict__ order) {
#pragma clang fp contract(off)
    using Slot = typename std::conditional<SMEM, uint16_t, uint32_t>::type;
    constexpr Slot kEmptySlot = (Slot)~(Slot)0;
    constexpr int ROWS = 4;  // rows rescanned at a time
    __shared__ WaveBest<T> wb[16], wa[16];     // a merge's nearest pair; row a
    __shared__ WaveBest<T> rb_[2][ROWS][16];   // rescanned rows, two sets taken in turn
    __shared__ int nlist[2];
    extern __shared__ __align__(16) char lds[];
    const int t = blockIdx.x;
    T *Dm = D + (int64_t)t * N * N;
    char *w = ws + (size_t)t * ws_stride;
    const size_t a4 = 256 * (((size_t)N * 4 + 255) / 256);
    const size_t aT = 256 * (((size_t)N * sizeof(T) + 255) / 256);
    int32_t *size = reinterpret_cast<int32_t *>(w + a4 + aT);
    int32_t *id = reinterpret_cast<int32_t *>(w + 2 * a4 + aT);
    int32_t *spare = reinterpret_cast<int32_t *>(w + 3 * a4 + aT);
    Slot *nn, *list;
    T *nd;
    const int tid = threadIdx.x, nth = blockDim.x;
    const int lane = tid & 63, wave = uniform(tid >> 6), nwaves = uniform(nth >> 6);
    if constexpr (SMEM) {
        const size_t sT = 16 * (((size_t)N * sizeof(T) + 15) / 16);
        const size_t s2 = 16 * (((size_t)N * 2 + 15) / 16);
        nd = reinterpret_cast<T *>(lds);
        nn = reinterpret_cast<Slot *>(lds + sT);
        list = reinterpret_cast<Slot *>(lds + sT + s2);
        const int32_t *gnn = reinterpret_cast<const int32_t *>(w);
        const T *gnd = reinterpret_cast<const T *>(w + a4);
        for (int k = tid; k < N; k += nth) {
            nn[k] = (Slot)gnn[k];
            nd[k] = gnd[k];
        }
    } else {
        nn = reinterpret_cast<Slot *>(w);
        nd = reinterpret_cast<T *>(w + a4);
        list = reinterpret_cast<Slot *>(spare);
    }
    auto barrier = [&]() __attribute__((always_inline)) {
        if constexpr (SMEM) local_barrier();
        else __syncthreads();
    };
    // the first of the workgroup's wave bests at `from`; every wave gets it
    auto first_of = [&](const WaveBest<T> *from, Best<T> &r, bool &mine) __attribute__((always_inline)) {
        Best<T> c;
        if (lane < nwaves) {
            c.key = from[lane].key;
            c.slot = from[lane].slot;
        }
        r = wave_best(c, mine);
    };
    double *Zm = Z + (int64_t)t * (N - 1) * 4;
    for (int k = tid; k < N; k += nth) {
        size[k] = 1;
        id[k] = k;
    }
    if (tid == 0) nlist[0] = nlist[1] = 0;
    __syncthreads();
    for (int m = 0; m + 1 < N; ++m) {
        // the first slot at the smallest nd
        Best<T> c;
        bool mine;
        for (int i = tid; i < N; i += nth)
            if (nn[i] != kEmptySlot) c.take(order_key(nd[i]), (uint32_t)i);
        c = wave_best(c, mine);
        if (lane == 0) wb[wave] = WaveBest<T>{c.key, c.slot, (T)0};
        __syncthreads();  // also: the last merge's stores to D, size and id
        first_of(wb, c, mine);
        // (two occupied slots always give a pair; the checks keep every index
        // below in range whatever D holds)
        if (c.slot >= (uint32_t)N) break;
        const int i0 = (int)c.slot, j0 = (int)nn[i0];
        const int a = i0 < j0 ? i0 : j0, b = i0 < j0 ? j0 : i0;
        if (b <= a || b >= N) break;
        const T dmin = nd[i0];
        const int na = size[a], nb = size[b];
        const int ida = tid == 0 ? id[a] : 0, idb = tid == 0 ? id[b] : 0;
        const T fa = (T)na, fb = (T)nb, fn = (T)(na + nb);
        // Rows whose nearest slot was a or b are listed for a rescan. The list
        // needs local memory only, so the first listed rows are read together
        // with rows a and b: one round trip to memory in place of two.
        T *ra = Dm + (int64_t)a * N;
        const T *rb = Dm + (int64_t)b * N;
        int *const nl = &nlist[m & 1];
        constexpr int U = sizeof(T) == 4 ? 4 : 2;  // slots of a thread read ahead
        T xa[U], xb[U], x0[ROWS][U];
        bool on[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = tid + u * nth;
            on[u] = q < N && nn[q < N ? q : 0] != kEmptySlot && q != a && q != b;
            xa[u] = on[u] ? ra[q] : (T)0;
            xb[u] = on[u] ? rb[q] : (T)0;
        }
        for (int k = tid; k < N; k += nth) {
            const Slot j = nn[k];
            if (j != kEmptySlot && k != a && k != b && ((int)j == a || (int)j == b))
                list[atomicAdd(nl, 1)] = (Slot)k;
        }
        barrier();
        const int nf = *nl;
        int row[ROWS];
        auto rows_of = [&](int f0) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) row[r] = (int)list[f0 + r < nf ? f0 + r : f0];
        };
        if (nf > 0) {
            rows_of(0);
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    x0[r][u] = on[u] ? Dm[(int64_t)row[r] * N + tid + u * nth] : (T)0;
        }
        // row and column a of the merged cluster; a listed row's nd then holds its
        // new distance to a, the others compare with it
        Best<T> ca;
        T da = (T)0;
        auto update = [&](int k, T va, T vb) __attribute__((always_inline)) {
            const T x = fa * va;
            const T y = fb * vb;
            const T s = x + y;
            const T d = s / fn;
            ra[k] = d;
            Dm[(int64_t)k * N + a] = d;
            const int j = (int)nn[k];
            if (j == a || j == b || before(d, a, nd[k], j)) {
                nn[k] = (Slot)a;
                nd[k] = d;
            }
            const auto key = order_key(d);
            if (key < ca.key) {
                ca.key = key;
                ca.slot = (uint32_t)k;
                da = d;
            }
        };
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (on[u]) update(tid + u * nth, xa[u], xb[u]);
        for (int k = tid + U * nth; k < N; k += nth)
            if (nn[k] != kEmptySlot && k != a && k != b) update(k, ra[k], rb[k]);
        {
            const Best<T> r = wave_best(ca, mine);
            if (mine) wa[wave].d = da;
            if (lane == 0) {
                wa[wave].key = r.key;
                wa[wave].slot = r.slot;
            }
        }
        if (tid == 0) {
            Zm[4 * m + 0] = (double)(ida < idb ? ida : idb);
            Zm[4 * m + 1] = (double)(ida < idb ? idb : ida);
            Zm[4 * m + 2] = (double)dmin;
            Zm[4 * m + 3] = (double)(na + nb);
            size[a] = na + nb;
            id[a] = N + m;
            nlist[(m + 1) & 1] = 0;
        }
        // rescan the listed rows, slot a apart (its distance is in nd)
        for (int f0 = 0, set = 0; f0 < nf; f0 += ROWS, set ^= 1) {
            Best<T> cr[ROWS];
            T dr[ROWS];
            if (f0 > 0) rows_of(f0);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) dr[r] = (T)0;
            auto scan = [&](int q, const T (&x)[ROWS]) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const auto key = order_key(x[r]);
                    if (q != row[r] && key < cr[r].key) {
                        cr[r].key = key;
                        cr[r].slot = (uint32_t)q;
                        dr[r] = x[r];
                    }
                }
            };
            int q = tid;
            if (f0 == 0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    T x[ROWS];
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) x[r] = x0[r][u];
                    if (on[u]) scan(tid + u * nth, x);
                }
                q += U * nth;
            }
#pragma unroll 2
            for (; q < N; q += nth) {
                if (nn[q] == kEmptySlot || q == a || q == b) continue;
                T x[ROWS];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) x[r] = Dm[(int64_t)row[r] * N + q];
                scan(q, x);
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const Best<T> best = wave_best(cr[r], mine);
                if (mine) rb_[set][r][wave].d = dr[r];
                if (lane == 0) {
                    rb_[set][r][wave].key = best.key;
                    rb_[set][r][wave].slot = best.slot;
                }
            }
            barrier();
            for (int r = wave; r < ROWS; r += nwaves) {
                if (f0 + r >= nf) break;
                Best<T> best;
                first_of(rb_[set][r], best, mine);
                const int k2 = (int)list[f0 + r];
                const auto key = order_key(nd[k2]);
                const bool keep = key < best.key || (key == best.key && (uint32_t)a < best.slot);
                if (mine && !keep) {
                    nn[k2] = (Slot)best.slot;
                    nd[k2] = rb_[set][r][lane].d;
                }
            }
        }
        if (nf == 0) barrier();
        if (wave == nwaves - 1) {  // the nearest slot of the merged row
            Best<T> r;
            first_of(wa, r, mine);
            if (mine) {
                nn[a] = (Slot)r.slot;
                nd[a] = wa[lane].d;
            }
            if (lane == 0) nn[b] = kEmptySlot;
        }
        barrier();
    }
    // Leaf order: depth first from the last merge, the smaller id first. The
    // first leaf of merge m's cluster stands at first[m]; taken from the last
    // merge down, each gives its two parts their first positions. One wave
    // reads 64 merges at a time (their parts and the size of the first part)
    // and steps through them.
    if (!order) return;
    int32_t *ord = order + (int64_t)t * N;
    int32_t *first = spare;
    __syncthreads();
    if (wave != 0) return;
    if (N == 1) {
        if (lane == 0) ord[0] = 0;
        return;
    }
    if constexpr (SMEM) first = reinterpret_cast<int32_t *>(lds);
    if (lane == 0) first[N - 2] = 0;
    for (int m1 = N - 2; m1 >= 0; m1 -= 64) {
        const int m = m1 - lane;
        // ids in Z are below 2N - 1 and those of merge m below N + m; the
        // checks only guard the indices
        int c0 = 0, c1 = 0, s0 = 1;
        if (m >= 0) {
            const double *z = Zm + 4 * (int64_t)m;
            c0 = (int)z[0];
            c1 = (int)z[1];
            if (c0 < 0 || c0 >= N + m) c0 = 0;
            if (c1 < 0 || c1 >= N + m) c1 = 0;
            if (c0 >= N) s0 = (int)Zm[4 * (int64_t)(c0 - N) + 3];
        }
        const int cntm = m1 + 1 < 64 ? m1 + 1 : 64;
        for (int q = 0; q < cntm; ++q) {
            const int p0 = __builtin_amdgcn_readlane(c0, q), p1 = __builtin_amdgcn_readlane(c1, q);
            const int n0 = __builtin_amdgcn_readlane(s0, q);
            if (lane < 2) {
                const int part = lane == 0 ? p0 : p1;
                const int at = *(volatile int32_t *)&first[m1 - q] + (lane == 0 ? 0 : n0);
                if (part >= N) *(volatile int32_t *)&first[part - N] = at;
                else if (at >= 0 && at < N) ord[at] = part;
            }
        }
    }
}

size_t linkage_workspace_bytes(int32_t N, int32_t T, int is_f64) {
    const size_t a4 = 256 * (((size_t)N * 4 + 255) / 256);
    const size_t aT = 256 * (((size_t)N * (is_f64 ? 8 : 4) + 255) / 256);
    const size_t a1 = 256 * (((size_t)N + 255) / 256);
    return (size_t)T * (4 * a4 + aT + a1);
}

namespace {

// Local memory a workgroup may allocate on the current device (0 if the
// runtime does not say), asked once per device.
size_t max_group_lds() {
    static std::mutex mu;
    static int known[64] = {};
    static size_t bytes[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    std::lock_guard<std::mutex> lock(mu);
    if (!known[dev]) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
            v = 0;
        bytes[dev] = v > 0 ? (size_t)v : 0;
        known[dev] = 1;
    }
    return bytes[dev];
}

template <class T>
hipError_t launch_linkage_t(T *D, int32_t N, int32_t T_, double *Z, int32_t *order, char *w,
                            hipStream_t st) {
    const size_t stride = linkage_workspace_bytes(N, 1, sizeof(T) == 8);
    const int64_t rows = (int64_t)N * T_;
    const int64_t blocks = (rows + 3) / 4;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    if (N > 1)
        hipLaunchKernelGGL(linkage_init_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, st,
                           (const T *)D, N, T_, stride, w);
    // threads per merge workgroup: 512 up to N = 1,024 (4.70 us per merge at
    // N = 1,000 against 5.22 with 1,024: fewer waves meet at the barriers),
    // else 1,024 (N = 3,000: 6.90 against 8.72); or LS_LINKAGE_THREADS (a
    // multiple of 64 up to 1024)
    int threads = N <= 1024 ? 512 : 1024;
    if (const char *env = std::getenv("LS_LINKAGE_THREADS")) {
        const int v = std::atoi(env);
        if (v >= 64 && v <= 1024 && v % 64 == 0) threads = v;
    }
    // the static part of the kernel's local memory: 10 x 16 wave bests, two counts
    const size_t lds = linkage_lds_bytes(N, sizeof(T));
    const size_t fixed = 10 * 16 * sizeof(WaveBest<T>) + 64;
    if (lds + fixed <= max_group_lds() && N <= kLinkageLdsMaxN) {
        // the kernel's limit is one value of the process: set to all there is, so
        // that threads clustering different N do not lower it for each other
        hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void *>(&linkage_kernel<T, true>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)(max_group_lds() - fixed));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((linkage_kernel<T, true>), dim3(T_), dim3(threads), lds, st, D, N,
                           stride, w, Z, order);
    } else {
        hipLaunchKernelGGL((linkage_kernel<T, false>), dim3(T_), dim3(threads), 0, st, D, N,
                           stride, w, Z, order);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_linkage(void *D, int32_t N, int32_t T, int is_f64, double *Z, int32_t *order,
                          void *ws, hipStream_t st) {
    if (N < 1 || T < 1) return hipSuccess;
    char *w = static_cast<char *>(ws);
    if (is_f64) return launch_linkage_t<double>((double *)D, N, T, Z, order, w, st);
    return launch_linkage_t<float>((float *)D, N, T, Z, order, w, st);
}

// ---------------------------------------------------------------------------
// Standardised half-distance rows (section 2.2): row (k, r) at E + k ts +
// r rs, recipient i = recips[r]; over the donors j != i, z = (e - mean) / sd
// with the population deviation (divisor N - 1), accumulated in FP64 in a
// fixed order; z_i = 0; a row whose donor entries are all equal becomes 0.
// In place. One workgroup of 256 per row.
template <class X>
__global__ void __launch_bounds__(256)
standardise_kernel(X *E, const int32_t *__restrict__ recips, int32_t N, int64_t ts, int64_t rs) {
    __shared__ double part[4];
    __shared__ int diff[4];
    const int r = blockIdx.x;
    const int64_t k = blockIdx.y;
    const int i = recips[r];
    X *row = E + k * ts + (int64_t)r * rs;
    const int first = i == 0 ? 1 : 0;
    const X x0 = row[first];
    double s = 0.0;
    int neq = 0;
    for (int j = threadIdx.x; j < N; j += 256) {
        if (j == i) continue;
        const X x = row[j];
        s += (double)x;
        neq |= !(x == x0);
    }
    const int wave = threadIdx.x >> 6;
    s = wave_sum(s);
    const int any = __any(neq);
    if ((threadIdx.x & 63) == 0) {
        part[wave] = s;
        diff[wave] = any;
    }
    __syncthreads();
    const double mean = ((part[0] + part[1]) + (part[2] + part[3])) / (double)(N - 1);
    const bool equal = !(diff[0] | diff[1] | diff[2] | diff[3]);
    double v = 0.0;
    for (int j = threadIdx.x; j < N; j += 256) {
        if (j == i) continue;
        const double d = (double)row[j] - mean;
        v += d * d;
    }
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[wave] = v;
    __syncthreads();
    const double sd = sqrt(((part[0] + part[1]) + (part[2] + part[3])) / (double)(N - 1));
    for (int j = threadIdx.x; j < N; j += 256)
        row[j] = (j == i || equal) ? (X)0 : (X)(((double)row[j] - mean) / sd);
}

hipError_t launch_standardise(void *E, const int32_t *recips, int32_t R, int32_t T, int32_t N,
                              int64_t ts, int64_t rs, int is_f64, hipStream_t st) {
    if (R < 1 || T < 1 || N < 2) return hipSuccess;
    if (T > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)R, (unsigned)T);
    if (is_f64)
        hipLaunchKernelGGL(standardise_kernel<double>, grid, dim3(256), 0, st, (double *)E,
                           recips, N, ts, rs);
    else
        hipLaunchKernelGGL(standardise_kernel<float>, grid, dim3(256), 0, st, (float *)E, recips,
                           N, ts, rs);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fixed scratch of the allocation-free linkage entry point: a file-scope
// device array, one copy per GPU, held until the process ends. In host code
// its name is not a device address; the address of each GPU's copy comes
// from hipGetSymbolAddress with that GPU current, taken once per GPU on its
// first use and kept.
static __device__ __align__(256) char scratch[kLinkageScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void *scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t linkage_scratch(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace lsk
