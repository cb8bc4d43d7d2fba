// CG on small systems as one kernel: the matrix stays in registers, the direction in LDS.
//
// A solve of launch-separated kernels reads the whole matrix every iteration and pays two
// launch gaps and two reduction prologues (about 9 us) on top.  Where the matrix fits the
// register files (36 8-byte values a lane and node pass, 512 KB a CU), each workgroup
// keeps the rows of its nodes for the whole solve, and only the vector z and the sums cross
// the chip.  What bounds an iteration then is the two sums over the grid.  Time per
// iteration, separate kernels -> this one (point Jacobi; with random node numbers in
// brackets):
//   FP64, 3 dofs per node, N = 675: 11.5 -> 4.6 us [11.3 -> 4.5]; 12,675: 11.6 -> 6.1;
//         54,243: 15.4 -> 8.0; 91,875: 19.1 -> 9.4 [25.1 -> 13]
//   FP32, 91,875: 13.6 -> 7.9; 186,219: 19.9 -> 10.9 [30.3 -> 16]
//   FP32, 1 dof per node, 9,261: 14.5 -> 6.2; 64,000: 17.1 -> 9.1
#include <condition_variable>
#include <cstring>
#include <mutex>

#include "internal.h"
#include "lanes.h"

namespace fem {
namespace {

constexpr int kResThreads = 512;         // 8 wavefronts, two per SIMD: 256 registers each
constexpr int kResWaves = kResThreads / 64;
constexpr int kResGroups = kResThreads / 8;  // nodes taken at a time, 8 lanes each
constexpr int kResMaxDeg = 32;               // four neighbour blocks per lane
constexpr int kSlotWords = 8;                // a 64-byte line per workgroup (see grid_sum)
constexpr int kAllToAll = 160;               // more workgroups than this sum through workgroup 0
constexpr int kResItsPerLaunch = 1024;

template <typename T>
__device__ __forceinline__ void store_agent(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ T load_agent(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sums over all workgroups; also the grid's barrier.  Every workgroup stores its total to
// its own line and reads all lines, one per thread: no atomic updates, one store and one
// load across the chip.  A word holds half of an FP64 value and the number of the round
// (`epoch`), so it is valid by itself and no flag has to follow the data.  Lines alternate
// with the round's parity: a workgroup can be one round ahead of one that still reads,
// never two.  What bounds it is the trip through the fabric (1.5 us a round with 8
// workgroups) and, with many workgroups, their reads of all lines (3.2 us with 256), so
// above kAllToAll workgroup 0 alone reads them and hands everyone the total on a line of
// its own.  CG iteration with 240 workgroups (91,875 dofs, FP64): 10.9 us all to all,
// 9.4 through workgroup 0; with 148 workgroups 8.0 and 8.1, with 69 workgroups 6.8 and 7.8.
// 32-byte slots cost the FP32 solve of the same mesh 0.7 us an iteration, slots packed
// into shared lines 2 to 3 us; fences at agent scope (which write back and
// invalidate L2) in place of the write-through accesses 13 us a round.
//
// Vector data: what the workgroup stored with store_agent before the call (the wait below)
// is what the others read with load_agent after it.  The wait for lines is bounded by the
// clock; on false, every thread of the workgroup leaves the kernel.
template <int NV>
__device__ __forceinline__ bool grid_sum(unsigned long long *slots, unsigned epoch, long long limit,
                                         const double (&v)[NV], double (&tot)[NV]) {
    __shared__ double red[2][kResWaves][NV];
    __shared__ int got_all[kResWaves];
    const int t = threadIdx.x, wave = t / 64, G = gridDim.x;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const double s = wave_sum(v[c]);
        if ((t & 63) == 0) red[0][wave][c] = s;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's vector stores have arrived
    __syncthreads();
    unsigned long long *buf = slots + size_t(epoch & 1) * kSlotWords * G;
    const unsigned long long tag = static_cast<unsigned long long>(epoch) << 32;
    if (t < NV) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kResWaves; ++w) s += red[0][w][t];
        const unsigned long long b = __builtin_bit_cast(unsigned long long, s);
        store_agent(buf + kSlotWords * blockIdx.x + 2 * t, tag | (b & 0xffffffffu));
        store_agent(buf + kSlotWords * blockIdx.x + 2 * t + 1, tag | (b >> 32));
    }
    // one value set (2 NV words at `w0`), bounded in time
    auto wait_for = [&](const unsigned long long *w0, double (&s)[NV]) -> bool {
        const long long t0 = wall_clock64();
        for (;;) {
            unsigned long long w[2 * NV];
            bool all = true;
#pragma unroll
            for (int c = 0; c < 2 * NV; ++c) w[c] = load_agent(w0 + c);
#pragma unroll
            for (int c = 0; c < 2 * NV; ++c) all &= unsigned(w[c] >> 32) == epoch;
            if (all) {
#pragma unroll
                for (int c = 0; c < NV; ++c)
                    s[c] = __builtin_bit_cast(double, (w[2 * c + 1] << 32) | (w[2 * c] & 0xffffffffu));
                return true;
            }
            if (wall_clock64() - t0 > limit) return false;
        }
    };
    double s[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) s[c] = 0.0;
    const bool relay = G > kAllToAll;
    unsigned long long *back = slots + size_t(2 + (epoch & 1)) * kSlotWords * G;
    bool ok = true;
    if (!relay || blockIdx.x == 0) {
        const bool got = t < G ? wait_for(buf + kSlotWords * t, s) : true;
        const bool wave_got = __all(got);
#pragma unroll
        for (int c = 0; c < NV; ++c) s[c] = wave_sum(s[c]);
        if ((t & 63) == 0) {
#pragma unroll
            for (int c = 0; c < NV; ++c) red[1][wave][c] = s[c];
            got_all[wave] = wave_got;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NV; ++c) tot[c] = 0.0;
#pragma unroll
        for (int w = 0; w < kResWaves; ++w) {
#pragma unroll
            for (int c = 0; c < NV; ++c) tot[c] += red[1][w][c];
            ok &= got_all[w] != 0;
        }
        if (relay && ok && t < G) {
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                const unsigned long long b = __builtin_bit_cast(unsigned long long, tot[c]);
                store_agent(back + kSlotWords * t + 2 * c, tag | (b & 0xffffffffu));
                store_agent(back + kSlotWords * t + 2 * c + 1, tag | (b >> 32));
            }
        }
    } else {
        if (t == 0) {
            got_all[0] = wait_for(back + kSlotWords * blockIdx.x, s);
#pragma unroll
            for (int c = 0; c < NV; ++c) red[1][0][c] = s[c];
        }
        __syncthreads();
        ok = got_all[0] != 0;
#pragma unroll
        for (int c = 0; c < NV; ++c) tot[c] = red[1][0][c];
    }
    return ok;
}

template <typename T, typename TV>
struct ResidentArgs {
    int64_t Nn;
    const int64_t *node_ptr;
    const int32_t *node_nb;
    const TV *values;
    const T *b, *dinv;
    T *x, *r, *p, *z;
    KrylovScalars *sc;
    unsigned long long *slots;
    unsigned epoch;    // first round number of this launch
    int chunk, cap;    // nodes per workgroup, capacity of its node list
    int bj;            // dinv holds node blocks
    int it0, it_end;   // iterations of this launch (it0 > 0: continue from x, r, p)
    double rtol;
    long long limit;   // clock ticks a workgroup waits for the others
};

// Workgroup b owns nodes [b chunk, (b + 1) chunk); eight lanes take one node (KN nodes one
// after the other), lane l neighbour blocks l, l + 8, l + 16, l + 24, whose values it keeps in
// registers.  Lanes 0..ND-1 of the eight own the node's entries of x and r.  LDS holds
// p for every node the workgroup's rows touch (`hid`: their numbers, found once by a bit
// map over all nodes), so the products gather from LDS and the update p = z + beta p
// reads each touched z once.  The steps and their order are those of the kernels in
// linalg.hip: the sums differ in their order only.
template <int ND, int KN, typename T, typename TV>
__global__ __launch_bounds__(kResThreads, 2) void k_cg_resident(ResidentArgs<T, TV> a) {
    extern __shared__ double dyn_lds[];
    __shared__ int wave_off[kResWaves];
    T *ps = reinterpret_cast<T *>(dyn_lds);
    int *hid = reinterpret_cast<int *>(ps + size_t(a.cap) * ND);
    const int W = int((a.Nn + 31) / 32);
    unsigned *bits = reinterpret_cast<unsigned *>(hid + a.cap);
    unsigned *pre = bits + W;
    const int t = threadIdx.x, l8 = t & 7, g8 = t / 8;
    const int64_t n0 = int64_t(blockIdx.x) * a.chunk;
    const int64_t n1 = n0 + a.chunk < a.Nn ? n0 + a.chunk : a.Nn;

    // ---- rows into registers, touched nodes into the bit map
    for (int w = t; w < W; w += kResThreads) bits[w] = 0;
    __syncthreads();
    TV v[KN][4][ND][ND];
    int pos[KN][4], po[KN];
    bool own[KN];
#pragma unroll
    for (int k = 0; k < KN; ++k) {
        const int64_t n = n0 + k * kResGroups + g8;
        const bool live = n < n1;
        const int64_t b0 = live ? a.node_ptr[n] : 0;
        const int deg = live ? int(a.node_ptr[n + 1] - b0) : 0;
        own[k] = live && l8 < ND;
        if (live && l8 == 0) atomicOr(&bits[n >> 5], 1u << (n & 31));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int l = l8 + 8 * j;
            const bool in = l < deg;
            const int m = in ? a.node_nb[b0 + l] : -1;
            pos[k][j] = m;
            if (in) atomicOr(&bits[m >> 5], 1u << (m & 31));
            const TV *vb = a.values + int64_t(ND) * ND * b0 + ND * l;
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int c = 0; c < ND; ++c) v[k][j][i][c] = in ? vb[int64_t(i) * ND * deg + c] : TV(0);
        }
    }
    __syncthreads();
    // ---- ranks of the marked nodes: position in LDS = number of marked nodes before
    int Hn;
    {
        const int per = (W + kResThreads - 1) / kResThreads;
        int mine = 0;
        for (int q = 0; q < per; ++q) {
            const int w = t * per + q;
            if (w < W) mine += __popc(bits[w]);
        }
        int incl = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if ((t & 63) >= o) incl += up;
        }
        if ((t & 63) == 63) wave_off[t / 64] = incl;
        __syncthreads();
        int base = incl - mine;
        Hn = 0;
        for (int w = 0; w < kResWaves; ++w) {
            if (w < t / 64) base += wave_off[w];
            Hn += wave_off[w];
        }
        for (int q = 0; q < per; ++q) {
            const int w = t * per + q;
            if (w >= W) break;
            pre[w] = base;
            unsigned bw = bits[w];
            while (bw) {
                const int bit = __ffs(bw) - 1;
                bw &= bw - 1;
                hid[base++] = 32 * w + bit;  // (at most cap: chunk nodes of at most max_deg neighbours)
            }
        }
    }
    __syncthreads();
    auto rank = [&](int64_t m) { return int(pre[m >> 5]) + __popc(bits[m >> 5] & ((1u << (m & 31)) - 1u)); };
#pragma unroll
    for (int k = 0; k < KN; ++k) {
        const int64_t n = n0 + k * kResGroups + g8;
        po[k] = own[k] ? rank(n) * ND + l8 : 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) pos[k][j] = pos[k][j] >= 0 ? rank(pos[k][j]) * ND : -1;
    }
    // ---- vectors
    T x[KN], r[KN], M[KN][ND];
#pragma unroll
    for (int k = 0; k < KN; ++k) {
        const int64_t d = ND * (n0 + k * kResGroups + g8) + l8;
        x[k] = own[k] && a.it0 > 0 ? a.x[d] : T(0);
        r[k] = own[k] ? (a.it0 > 0 ? a.r[d] : a.b[d]) : T(0);
#pragma unroll
        for (int c = 0; c < ND; ++c)
            M[k][c] = !own[k] ? T(0) : (a.bj ? a.dinv[ND * d + c] : (c == 0 ? a.dinv[d] : T(0)));
    }
    // z = M r of the owned entries, to memory for the others; sums of r z and r r
    auto precondition = [&](double (&dots)[2]) {
        dots[0] = dots[1] = 0.0;
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            T z = M[k][0] * r[k];
            if constexpr (ND == 3) {
                if (a.bj)  // r of lanes 0, 1, 2 of the quad
                    z = M[k][0] * dpp_read<0x00>(r[k]) + M[k][1] * dpp_read<0x55>(r[k]) + M[k][2] * dpp_read<0xAA>(r[k]);
            }
            if (own[k]) {
                store_agent(a.z + ND * (n0 + k * kResGroups + g8) + l8, z);
                dots[0] += double(r[k]) * double(z);
                dots[1] += double(r[k]) * double(r[k]);
            }
        }
    };
    // p = z + beta p on all touched nodes
    auto direction = [&](bool first, T beta) {
        constexpr int U = 4;  // loads in flight per thread
        for (int e0 = t; e0 < Hn * ND; e0 += U * kResThreads) {
            T z[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int e = e0 + q * kResThreads;
                const int ec = e < Hn * ND ? e : e0;
                z[q] = load_agent(a.z + int64_t(ND) * hid[ec / ND] + ec % ND);
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int e = e0 + q * kResThreads;
                if (e < Hn * ND) ps[e] = first ? z[q] : z[q] + beta * ps[e];
            }
        }
        __syncthreads();
    };
    unsigned epoch = a.epoch;
    double rho, bnorm2, rnorm2, tol2;
    int its = a.it0, converged = 0, breakdown = 0;
    if (a.it0 == 0) {
        double dots[2], tot[2];
        precondition(dots);
        if (!grid_sum<2>(a.slots, epoch++, a.limit, dots, tot)) {
            if (t == 0) a.sc->aborted = int(a.epoch);
            return;
        }
        rho = tot[0];
        bnorm2 = rnorm2 = tot[1];
        tol2 = a.rtol * a.rtol * bnorm2;
        breakdown = isfinite(tot[1]) ? 0 : 2;
        converged = tot[1] == 0.0;
        direction(true, T(0));
    } else {
        rho = a.sc->rho;  // (rewritten by workgroup 0 after the first round only)
        bnorm2 = a.sc->bnorm2;
        rnorm2 = a.sc->rnorm2;
        tol2 = a.sc->tol2;
        for (int e = t; e < Hn * ND; e += kResThreads) ps[e] = a.p[int64_t(ND) * hid[e / ND] + e % ND];
        __syncthreads();
    }
    // ---- iterations
    for (int it = a.it0; it < a.it_end && !converged && !breakdown; ++it) {
        T q[KN], p[KN];
        double dot[1] = {0.0}, pq[1];
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            T acc[ND];
#pragma unroll
            for (int i = 0; i < ND; ++i) acc[i] = T(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                T pm[ND];
                const int at = pos[k][j] >= 0 ? pos[k][j] : 0;
#pragma unroll
                for (int c = 0; c < ND; ++c) pm[c] = ps[at + c];
#pragma unroll
                for (int i = 0; i < ND; ++i)
#pragma unroll
                    for (int c = 0; c < ND; ++c) acc[i] += T(v[k][j][i][c]) * (pos[k][j] >= 0 ? pm[c] : T(0));
            }
#pragma unroll
            for (int i = 0; i < ND; ++i) acc[i] = lane_sum8(acc[i]);
            q[k] = acc[0];
            if constexpr (ND == 3) q[k] = l8 == 1 ? acc[1] : (l8 == 2 ? acc[2] : acc[0]);
            p[k] = own[k] ? ps[po[k]] : T(0);
            if (own[k]) dot[0] += double(p[k]) * double(q[k]);
        }
        if (!grid_sum<1>(a.slots, epoch++, a.limit, dot, pq)) {
            if (t == 0) a.sc->aborted = int(a.epoch);
            return;
        }
        if (!(pq[0] > 0.0) || !isfinite(pq[0])) {  // CG needs (p, K p) > 0
            breakdown = 1;
            break;
        }
        const T al = T(rho / pq[0]);
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            x[k] += al * p[k];
            r[k] -= al * (own[k] ? q[k] : T(0));
        }
        double dots[2], tot[2];
        precondition(dots);
        if (!grid_sum<2>(a.slots, epoch++, a.limit, dots, tot)) {
            if (t == 0) a.sc->aborted = int(a.epoch);
            return;
        }
        its = it + 1;
        rnorm2 = tot[1];
        if (!isfinite(tot[0]) || !isfinite(tot[1])) breakdown = 2;
        else if (tot[1] <= tol2) converged = 1;
        const T beta = T(tot[0] / rho);
        rho = tot[0];
        if (!converged && !breakdown) direction(false, beta);
    }
#pragma unroll
    for (int k = 0; k < KN; ++k) {
        if (!own[k]) continue;
        const int64_t d = ND * (n0 + k * kResGroups + g8) + l8;
        a.x[d] = x[k];
        a.r[d] = r[k];
        if (!converged && !breakdown) a.p[d] = ps[po[k]];
    }
    if (blockIdx.x == 0 && t == 0) {
        KrylovScalars *sc = a.sc;
        sc->rho = rho;
        sc->bnorm2 = bnorm2;
        sc->rnorm2 = rnorm2;
        sc->tol2 = tol2;
        sc->its = its;
        sc->converged = converged;
        sc->breakdown = breakdown;
    }
}

// Workgroups of resident solves on one device wait for one another, so all of them have to
// fit the device at once: a solve takes its share of the compute units here before the
// launch and gives it back when its kernel has ended (other threads' solves wait).
class ComputeUnits {
public:
    ComputeUnits(int device, int n, int total) : pool_(pool(device)), n_(n) {
        std::unique_lock<std::mutex> lk(pool_.m);
        pool_.cv.wait(lk, [&] { return pool_.used + n_ <= total; });
        pool_.used += n_;
    }
    ~ComputeUnits() {
        {
            std::lock_guard<std::mutex> lk(pool_.m);
            pool_.used -= n_;
        }
        pool_.cv.notify_all();
    }
    ComputeUnits(const ComputeUnits &) = delete;
    ComputeUnits &operator=(const ComputeUnits &) = delete;

private:
    struct Pool {
        std::mutex m;
        std::condition_variable cv;
        int used = 0;
    };
    static Pool &pool(int device) {
        static Pool pools[64];
        return pools[device & 63];
    }
    Pool &pool_;
    int n_;
};

struct ResidentPlan {
    int kn = 0, grid = 0, chunk = 0, cap = 0;
    size_t lds = 0;
};

// Nodes per 8-lane group (kn) and workgroups: at most what the registers hold (144 of 256
// with values), and few enough touched nodes for the LDS whatever the numbering.  Few
// workgroups sum faster, many have shorter rows of work: kn = 1 up to 16 workgroups, else
// the largest (FP64, 3 dofs per node: N = 4,131, 22 workgroups 5.8 us an iteration, 11 5.7;
// 26,877: 7.7 with kn = 1, 7.1 with 2; one dof per node, 28,611 dofs: 12.0 us with kn = 2,
// 10.4 with 4; FP64, 729: 3% better with kn = 1 than with 4).
template <int ND, typename T, typename TV>
ResidentPlan resident_plan(const fem_handle *h) {
    constexpr int kMax = ND == 1 ? 4 : (sizeof(T) == 4 ? 4 : 2);
    const Graph &g = h->g;
    ResidentPlan p;
    if (g.max_deg < 1 || g.max_deg > kResMaxDeg || h->cg_slots == nullptr || h->cg_slots_off) return p;
    for (int kn = 1; kn <= kMax; kn *= 2) {
        const int64_t per = int64_t(kn) * kResGroups;
        const int64_t grid = (g.Nn + per - 1) / per;
        if (grid > h->num_cus) continue;
        const int64_t chunk = (g.Nn + grid - 1) / grid;
        const int64_t cap = (std::min<int64_t>(chunk * g.max_deg, g.Nn) + 1) / 2 * 2;
        const size_t lds = size_t(cap) * (ND * sizeof(T) + sizeof(int)) + size_t((g.Nn + 31) / 32) * 8;
        if (lds + 1024 > size_t(h->lds_bytes)) break;
        p.kn = kn;
        p.grid = int(grid);
        p.chunk = int(chunk);
        p.cap = int(cap);
        p.lds = lds;
        if (grid <= 16) break;
    }
    return p;
}

template <int ND, int KN, typename T, typename TV>
void resident_launch(const ResidentPlan &pl, const ResidentArgs<T, TV> &a, hipStream_t s) {
    if (pl.lds > 65536)
        FEM_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_cg_resident<ND, KN, T, TV>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, int(pl.lds)));
    hipLaunchKernelGGL((k_cg_resident<ND, KN, T, TV>), dim3(pl.grid), dim3(kResThreads), pl.lds, s, a);
    FEM_HIP(hipGetLastError());
}

template <int ND, typename T, typename TV>
bool resident_solve(fem_handle *h, const KrylovVecs<T> &k, const TV *values, const T *b, double rtol, int64_t max_its,
                    KrylovScalars &hs, hipStream_t s) {
    const ResidentPlan pl = resident_plan<ND, T, TV>(h);
    if (pl.kn == 0) return false;
    const Graph &g = h->g;
    ResidentArgs<T, TV> a{g.Nn,       g.node_ptr, g.node_nb, values, b,   k.dinv, k.x, k.r, k.p, k.rh, k.sc,
                          h->cg_slots, 0,          pl.chunk,  pl.cap, k.bj, 0,      0,   rtol, 100ll * h->clock_khz};
    ComputeUnits share(h->device, pl.grid, h->num_cus);
    for (;;) {
        a.it_end = int(std::min<int64_t>(max_its, int64_t(a.it0) + kResItsPerLaunch));
        if (h->cg_epoch > 0x70000000u) {  // round numbers of the far past must not come up again
            FEM_HIP(hipMemsetAsync(h->cg_slots, 0, resident_slots_bytes(h), s));
            h->cg_epoch = 0;
        }
        a.epoch = h->cg_epoch + 1;
        h->cg_epoch += 2 * kResItsPerLaunch + 8;
        if constexpr (ND == 1) {
            if (pl.kn == 1) resident_launch<1, 1>(pl, a, s);
            else if (pl.kn == 2) resident_launch<1, 2>(pl, a, s);
            else resident_launch<1, 4>(pl, a, s);
        } else {
            if (pl.kn == 1) resident_launch<3, 1>(pl, a, s);
            else if (pl.kn == 2) resident_launch<3, 2>(pl, a, s);
            else if constexpr (sizeof(T) == 4) resident_launch<3, 4>(pl, a, s);
        }
        FEM_HIP(hipMemcpyAsync(h->host_kry, k.sc, kScalarsHostBytes, hipMemcpyDeviceToHost, s));
        FEM_HIP(hipStreamSynchronize(s));
        std::memcpy(&hs, h->host_kry, kScalarsHostBytes);
        if (hs.aborted == int(a.epoch)) {
            // the workgroups were not all running together (compute units held by other
            // work): this solve and the handle's later ones take the separate kernels
            h->cg_slots_off = true;
            return false;
        }
        if (hs.converged || hs.breakdown || hs.its >= max_its) return true;
        a.it0 = hs.its;
    }
}

}  // namespace

size_t resident_slots_bytes(const fem_handle *h) {
    return size_t(4) * kSlotWords * h->num_cus * sizeof(unsigned long long);
}

template <typename T>
bool kry_cg_resident(fem_handle *h, const KrylovVecs<T> &k, const T *b, double rtol, int64_t max_its,
                     KrylovScalars &hs, hipStream_t s) {
    if (k.layout != LAYOUT_CSR || h->g.N == 0) return false;
    if constexpr (sizeof(T) == 8) {
        if (k.A32)
            return h->g.nd == 1 ? resident_solve<1, T, float>(h, k, k.A32, b, rtol, max_its, hs, s)
                                : resident_solve<3, T, float>(h, k, k.A32, b, rtol, max_its, hs, s);
    }
    return h->g.nd == 1 ? resident_solve<1, T, T>(h, k, k.A, b, rtol, max_its, hs, s)
                        : resident_solve<3, T, T>(h, k, k.A, b, rtol, max_its, hs, s);
}

template bool kry_cg_resident<float>(fem_handle *, const KrylovVecs<float> &, const float *, double, int64_t,
                                     KrylovScalars &, hipStream_t);
template bool kry_cg_resident<double>(fem_handle *, const KrylovVecs<double> &, const double *, double, int64_t,
                                      KrylovScalars &, hipStream_t);

}  // namespace fem
