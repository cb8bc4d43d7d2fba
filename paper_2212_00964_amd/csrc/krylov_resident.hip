// Krylov solves on small and middle systems as one kernel: as much of the matrix as fits
// stays in registers, the gathered vectors in LDS.
//
// A solve of launch-separated kernels reads the whole matrix every iteration and pays two
// to five launch gaps and reduction prologues (9 to 18 us) on top.  Here each workgroup (one
// per CU) keeps the rows of up to KN nodes per 8-lane group in registers for the whole
// solve (36 values a lane and node: 144 of 256 registers), as many more as fit in LDS, and
// reads the rest again in every product; only the vectors and the sums cross the chip.
// What bounds an iteration is the sums over the grid (two for CG, three for BiCGSTAB: 2.8 us
// each at 240 workgroups), and beyond the registers the latency of the rows read again (two
// wavefronts per SIMD hide little of it; asking for them before the register passes, or
// two blocks ahead in FP64, spills registers and costs 5 us more).
// Time per iteration on box meshes, separate kernels -> this one, us (rows beyond the
// registers from 32,768 nodes on with 8-byte values, 65,536 with 4-byte ones or one dof):
//   CG, FP64        N = 675 11.5 -> 5.4, 12,675 11.6 -> 6.3, 91,875 18.7 -> 9.4,
//                   212,355 31.8 -> 19.5, 260,925 36.8 -> 24.5
//   CG, FP32        91,875 13.5 -> 8.2, 186,219 20.0 -> 10.3, 260,925 23.4 -> 14.6
//   CG, FP32, one dof per node      9,261 13.1 -> 5.5, 64,000 16.5 -> 8.3, 250,047 30.0 -> 14.7
//   BiCGSTAB, FP64  3,993 17.4 -> 10.1, 98,304 37.7 -> 18.1, 206,763 59.2 -> 43.7
//   BiCGSTAB, FP32 values under FP64 vectors      46,875 23.1 -> 18.3, 192,000 40.9 -> 24.4,
//                   206,763 43.4 -> 30.4, 255,552 47.8 -> 38.0
//   BiCGSTAB, FP32  98,304 28.4 -> 16.7, 206,763 41.7 -> 24.0
// With random node numbers a workgroup touches more nodes: CG, FP64, 91,875 25.0 -> 12.3;
// where they do not fit the LDS the separate kernels run (CG, FP64 from 186,219).
#include <algorithm>
#include <condition_variable>
#include <mutex>

#include "bicg_rules.h"
#include "internal.h"
#include "lanes.h"

namespace fem {
namespace {

constexpr int kResThreads = 512;         // 8 wavefronts, two per SIMD: 256 registers each
constexpr int kResWaves = kResThreads / 64;
constexpr int kResGroups = kResThreads / 8;  // nodes taken at a time, 8 lanes each
constexpr int kResMaxDeg = 32;               // four neighbour blocks per lane
constexpr int kResDofs = 2;                  // owned dofs per thread
constexpr int kSlotWords = 8;                // a 64-byte line per workgroup (see grid_sum)
constexpr int kAllToAll = 160;               // more workgroups than this sum through workgroup 0
constexpr int kResItsPerLaunch = 1024;
constexpr int kResMaxBackoff = 64;           // solves skipped after a give-up, at most
enum : int { kGaveUp = 1, kMisfit = 2 };     // why a launch left the solve undone
constexpr size_t kResStaticLds = 1024;       // the sums' arrays

template <typename T>
__device__ __forceinline__ void store_agent(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ T load_agent(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A value that is the same in all lanes, moved to scalar registers (what comes out of LDS or
// of FP64 arithmetic sits in vector registers otherwise, and those are what is short here).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uniform(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readfirstlane(int(b & 0xffffffffu));
    const unsigned hi = __builtin_amdgcn_readfirstlane(int(b >> 32));
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
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
// invalidate L2) in place of the write-through accesses 10 to 17 us a round.
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
#pragma unroll
    for (int c = 0; c < NV; ++c) tot[c] = uniform(tot[c]);
    return uniform(int(ok)) != 0;
}

template <typename T, typename TV>
struct ResidentArgs {
    int64_t Nn;
    const int64_t *node_ptr;
    const int32_t *node_nb;
    const TV *values;
    const T *b, *dinv;
    T *x, *r, *p, *v, *t, *rh;  // CG exchanges z in rh; BiCGSTAB v and t
    KrylovScalars *sc;       // for the next launch of the same solve
    KrylovScalars *host;     // pinned: what the host reads when the kernel has ended
    unsigned long long *slots;
    unsigned epoch;    // first round number of this launch
    int chunk;         // nodes per workgroup
    int lds;           // bytes of LDS
    int check_fit;     // whether the touched nodes may not fit it
    int bj;            // dinv holds node blocks
    int it0, it_end;   // iterations of this launch (it0 > 0: continue from x, r, p ...)
    double rtol;
    long long limit;   // clock ticks a workgroup waits for the others
};

// Neighbour block j of lane l8 of a node's eight, and the sum over the eight: with the lane's
// blocks added in pairs (0, 1) and (2, 3), a row is summed in the order of the separate
// kernels' 32 lanes (group32_sum) and rounds the same.
__device__ __forceinline__ int lane_block(int l8, int j) { return 16 * (j & 1) + (j < 2 ? l8 : 15 - l8); }
template <typename T>
__device__ __forceinline__ T row_sum8(T v) {
    v += dpp_read<kDppHalfMirror>(v);
    v += dpp_read<kDppXor2>(v);
    v += dpp_read<kDppXor1>(v);
    return v;
}

// The rows of workgroup b: nodes [b chunk, (b + 1) chunk).  Eight lanes take one node, four of its
// neighbour blocks each (lane_block).  The first KN passes over the workgroup's
// nodes have their values in registers; of the others (MORE) as many as fit stay in LDS
// and the rest are read from memory in every product.  Touched nodes are numbered for LDS: the workgroup's own first, then the
// others in ascending order (found once by a bit map over all nodes; `hid` lists the
// others), then one whose entries stay zero, for the lanes without a block.
template <int ND, int KN, bool MORE, typename T, typename TV>
struct ResidentRows {
    // owned dofs per thread
    static constexpr int kDofs = MORE ? kResDofs : (KN * kResGroups * ND + kResThreads - 1) / kResThreads;
    static constexpr int kFirst = KN * kResGroups;  // nodes in registers
    static_assert(sizeof(double) >= sizeof(TV), "LDS regions are laid out in doubles");
    TV v[KN][4][ND][ND];
    unsigned pos[KN][2];  // LDS index of the neighbour's first entry, two to a word
    const TV *values;
    const int32_t *nb;
    int64_t n0, b0;      // first node and first block
    int cnt, Hn;         // own and touched nodes
    int in_lds;          // nodes after the first kFirst with values in LDS
    int rest;            // their first block
    int *hid, *rowp;
    unsigned *bits;
    uint16_t *pre, *npos;
    TV *lv;

    __device__ __forceinline__ int where(int m) const {
        const unsigned o = unsigned(m - int(n0));
        if (o < unsigned(cnt)) return int(o) * ND;
        return (cnt + int(pre[m >> 5]) + __popc(bits[m >> 5] & ((1u << (m & 31)) - 1u))) * ND;
    }

    // Loads the rows and numbers the touched nodes; takes its LDS from `lds` (8-byte
    // aligned) on and returns the bytes used.  Reads nothing it has not room for: false
    // in `fits` means that the touched nodes (`each` bytes each) do not fit a.lds bytes.
    __device__ __forceinline__ size_t setup(const ResidentArgs<T, TV> &a, char *lds, size_t fixed, size_t each,
                                            bool &fits) {
        __shared__ int wave_off[kResWaves];
        const int t = threadIdx.x, l8 = t & 7, g8 = t / 8;
        const int W = int((a.Nn + 31) / 32);
        bits = reinterpret_cast<unsigned *>(lds);
        rowp = reinterpret_cast<int *>(bits + W);
        hid = rowp + a.chunk + 1;
        values = a.values;
        nb = a.node_nb;
        n0 = int64_t(blockIdx.x) * a.chunk;
        cnt = int(n0 + a.chunk < a.Nn ? a.chunk : a.Nn - n0);
        b0 = a.node_ptr[n0];
        for (int w = t; w < W; w += kResThreads) bits[w] = 0;
        for (int i = t; i <= cnt; i += kResThreads) rowp[i] = int(a.node_ptr[n0 + i] - b0);
        __syncthreads();
        auto mark = [&](int m) {
            if (unsigned(m - int(n0)) >= unsigned(cnt)) atomicOr(&bits[m >> 5], 1u << (m & 31));
        };
        int nbm[KN][4];
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            const int ln = k * kResGroups + g8;
            const int s0 = ln < cnt ? rowp[ln] : 0, deg = ln < cnt ? rowp[ln + 1] - s0 : 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int l = lane_block(l8, j);
                nbm[k][j] = l < deg ? nb[b0 + s0 + l] : -1;
                if (l < deg) mark(nbm[k][j]);
                const TV *vb = values + int64_t(ND) * ND * (b0 + s0) + ND * l;
#pragma unroll
                for (int i = 0; i < ND; ++i)
#pragma unroll
                    for (int c = 0; c < ND; ++c) v[k][j][i][c] = l < deg ? vb[i * ND * deg + c] : TV(0);
            }
        }
        rest = uniform(MORE && kFirst < cnt ? rowp[kFirst] : rowp[cnt]);
        for (int i = rest + t; i < rowp[cnt]; i += kResThreads) mark(nb[b0 + i]);
        __syncthreads();
        // number of marked nodes before each word of the bit map
        const int per = (W + kResThreads - 1) / kResThreads;
        int mine = 0;
        for (int q = 0; q < per; ++q)
            if (t * per + q < W) mine += __popc(bits[t * per + q]);
        int incl = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if ((t & 63) >= o) incl += up;
        }
        if ((t & 63) == 63) wave_off[t / 64] = incl;
        __syncthreads();
        int base = incl - mine;
        Hn = cnt;
        for (int w = 0; w < kResWaves; ++w) {
            if (w < t / 64) base += wave_off[w];
            Hn += wave_off[w];
        }
        Hn = uniform(Hn);
        // LDS after hid: ranks, positions of the rows outside the registers; then the
        // caller's vectors (fixed + each bytes per touched node) and the rows kept in LDS
        size_t used = sizeof(unsigned) * W + sizeof(int) * (a.chunk + 1 + (Hn - cnt));
        pre = reinterpret_cast<uint16_t *>(lds + used);
        npos = pre + W;
        used += sizeof(uint16_t) * (W + (MORE ? uniform(rowp[cnt]) - rest : 0));
        used = (used + 7) / 8 * 8;
        const size_t vectors = (fixed + each * (Hn + 1) + 7) / 8 * 8;
        fits = used + vectors <= size_t(a.lds);
        in_lds = 0;
        if (!fits) return used;
        lv = reinterpret_cast<TV *>(lds + used + vectors);
        if constexpr (MORE) {
            const int room = int((size_t(a.lds) - used - vectors) / (sizeof(TV) * ND * ND));  // blocks
            if (kFirst < cnt)
                while (kFirst + in_lds < cnt && rowp[kFirst + in_lds + 1] - rest <= room) ++in_lds;
            in_lds = uniform(in_lds);
        }
        for (int q = 0; q < per; ++q) {
            const int w = t * per + q;
            if (w >= W) break;
            pre[w] = uint16_t(base);
            for (unsigned bw = bits[w]; bw; bw &= bw - 1, ++base) hid[base] = 32 * w + __ffs(bw) - 1;
        }
        __syncthreads();
        const int none = Hn * ND;
#pragma unroll
        for (int k = 0; k < KN; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned at = unsigned(nbm[k][j] >= 0 ? where(nbm[k][j]) : none);
                if (j % 2 == 0) pos[k][j / 2] = at;
                else pos[k][j / 2] |= at << 16;
            }
        if constexpr (MORE) {
            for (int i = rest + t; i < rowp[cnt]; i += kResThreads) npos[i - rest] = uint16_t(where(nb[b0 + i]));
            if (in_lds > 0) {
                const int n = ND * ND * (rowp[kFirst + in_lds] - rest);
                for (int i = t; i < n; i += kResThreads) lv[i] = values[int64_t(ND) * ND * (b0 + rest) + i];
            }
        }
        return used;
    }

    // out(local node, row value) in lanes 0..ND-1 of each group for y = A x, x in LDS.
    template <typename F>
    __device__ __forceinline__ void product(const T *x, F &&out) {
        const int l8 = threadIdx.x & 7, g8 = threadIdx.x / 8;
        auto finish = [&](int ln, T (&acc)[ND]) {
#pragma unroll
            for (int i = 0; i < ND; ++i) acc[i] = row_sum8(acc[i]);
            T q = acc[0];
            if constexpr (ND == 3) q = l8 == 1 ? acc[1] : (l8 == 2 ? acc[2] : acc[0]);
            if (ln < cnt && l8 < ND) out(ln, q);
        };
        // The products of a block.  (One chain of all 12 products of a lane left FP32 rows 8%
        // further off than the separate kernels', 25% with one dof per node at 42^3.)
        auto block = [&](T (&s)[ND], const TV (&w)[ND][ND], int at) {
            T xm[ND];
#pragma unroll
            for (int c = 0; c < ND; ++c) xm[c] = x[at + c];
#pragma unroll
            for (int i = 0; i < ND; ++i) {
                s[i] = T(0);
#pragma unroll
                for (int c = 0; c < ND; ++c) s[i] += T(w[i][c]) * xm[c];
            }
        };
        // a += b, not contracted with the products behind b
        auto add = [&](T (&a)[ND], const T (&b)[ND]) {
#pragma clang fp contract(off)
#pragma unroll
            for (int i = 0; i < ND; ++i) a[i] += b[i];
        };
        // The lane's block j of a node outside the registers (its blocks s0 .. s0 + deg) from `src`, the
        // values of the blocks from `from` on; zeros and the zero entry where there is none.
        auto load = [&](const TV *src, int from, int s0, int deg, int j, TV (&w)[ND][ND], int &at) {
            const int l = lane_block(l8, j);
            const bool in = l < deg;
            const TV *vb = src + int64_t(ND) * ND * (s0 - from) + ND * l;
            at = in ? int(npos[s0 + l - rest]) : Hn * ND;
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int c = 0; c < ND; ++c) w[i][c] = in ? vb[i * ND * deg + c] : TV(0);
        };
        // FP64 blocks of three dofs one at a time: two in flight spill registers
        constexpr bool kOne = ND * sizeof(TV) > 12;
        // acc += blocks j and j + 1
        auto pair = [&](T (&acc)[ND], const TV *src, int from, int s0, int deg, int j0) {
#pragma unroll 1
            for (int j = j0; j < j0 + 2; ++j) {
                TV w[ND][ND];
                T s[ND];
                int at;
                load(src, from, s0, deg, j, w, at);
                block(s, w, at);
                add(acc, s);
            }
        };
        auto row = [&](int ln, int end, int &s0, int &deg) {
            s0 = ln < end ? rowp[ln] : rest;
            deg = ln < end ? rowp[ln + 1] - s0 : 0;
        };
        const int s1 = kFirst + in_lds;  // first node read from memory
        const TV *mem = values + int64_t(ND) * ND * b0;
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            T acc[ND];
#pragma unroll
            for (int i = 0; i < ND; ++i) acc[i] = T(0);
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
                T s[2][ND];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if constexpr (sizeof(TV) < sizeof(T)) {
                        // converted here each time: out of the loop the FP64 values would
                        // take twice the registers
#pragma unroll
                        for (int i = 0; i < ND; ++i)
#pragma unroll
                            for (int c = 0; c < ND; ++c) asm volatile("" : "+v"(v[k][j + q][i][c]));
                    }
                    block(s[q], v[k][j + q], int(q ? pos[k][j / 2] >> 16 : pos[k][j / 2] & 0xffffu));
                }
                add(s[0], s[1]);
                add(acc, s[0]);
            }
            finish(k * kResGroups + g8, acc);
        }
        // (all lanes of a wavefront take every pass: the sums use all of them)
        if constexpr (MORE) {
#pragma unroll 1
            for (int l0 = kFirst; l0 < s1; l0 += kResGroups) {
                T acc[ND], acc2[ND];
#pragma unroll
                for (int i = 0; i < ND; ++i) acc[i] = acc2[i] = T(0);
                int ls, ld;
                row(l0 + g8, s1, ls, ld);
                if constexpr (kOne) {
                    pair(acc, lv, rest, ls, ld, 0);
                    pair(acc2, lv, rest, ls, ld, 2);
                    add(acc, acc2);
                } else {
#pragma unroll 1
                    for (int j = 0; j < 4; j += 2) {
                        T s[2][ND];
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            TV wl[ND][ND];
                            int al;
                            load(lv, rest, ls, ld, j + q, wl, al);
                            block(s[q], wl, al);
                            asm volatile("" ::: "memory");
                        }
                        add(s[0], s[1]);
                        add(acc, s[0]);
                    }
                }
                finish(l0 + g8 < s1 ? l0 + g8 : cnt, acc);
            }
#pragma unroll 1
            for (int l0 = s1; l0 < cnt; l0 += kResGroups) {
                T acc[ND], acc2[ND];
#pragma unroll
                for (int i = 0; i < ND; ++i) acc[i] = acc2[i] = T(0);
                int s0, deg;
                row(l0 + g8, cnt, s0, deg);
                if constexpr (kOne) {
                    pair(acc, mem, 0, s0, deg, 0);
                    pair(acc2, mem, 0, s0, deg, 2);
                    add(acc, acc2);
                } else {
#pragma unroll 1
                    for (int j = 0; j < 4; j += 2) {
                        T s[2][ND];
                        TV w[2][ND][ND];
                        int at[2];
                        load(mem, 0, s0, deg, j, w[0], at[0]);
                        load(mem, 0, s0, deg, j + 1, w[1], at[1]);
                        block(s[0], w[0], at[0]);
                        block(s[1], w[1], at[1]);
                        add(s[0], s[1]);
                        add(acc, s[0]);
                    }
                }
                finish(l0 + g8, acc);
            }
        }
    }

    // f(LDS entry, value of src) for every touched entry outside the workgroup, with
    // src written by the others through store_agent.
    template <typename F>
    __device__ __forceinline__ void gather(const T *src, F &&f) const {
        constexpr int U = 4;  // loads in flight per thread
        const int n = (Hn - cnt) * ND;
        for (int e0 = threadIdx.x; e0 < n; e0 += U * kResThreads) {
            T z[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int e = e0 + q * kResThreads, ec = e < n ? e : e0;
                z[q] = load_agent(src + int64_t(ND) * hid[ec / ND] + ec % ND);
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int e = e0 + q * kResThreads;
                if (e < n) f(cnt * ND + e, z[q]);
            }
        }
    }
};

// Returns whether all workgroups' touched nodes fit their LDS (asked only where they may
// not); otherwise the launch ends and the host takes the separate kernels.
template <typename T, typename TV>
__device__ __forceinline__ bool resident_fits(const ResidentArgs<T, TV> &a, bool fits, unsigned &epoch) {
    if (!a.check_fit) return true;
    const double miss[1] = {threadIdx.x == 0 && !fits ? 1.0 : 0.0};
    double tot[1];
    const bool ok = grid_sum<1>(a.slots, epoch++, a.limit, miss, tot);
    if (ok && tot[0] == 0.0) return true;
    if (threadIdx.x == 0 && (!ok || blockIdx.x == 0)) a.host->aborted = ok ? kMisfit : kGaveUp;
    return false;
}

// CG: the steps and their order are those of the kernels in linalg.hip; the sums differ in
// their order only.  LDS: p on the touched nodes, q on the owned ones.
template <int ND, int KN, bool MORE, typename T, typename TV>
__global__ __launch_bounds__(kResThreads, 2) void k_cg_resident(ResidentArgs<T, TV> a) {
    extern __shared__ double dyn_lds[];
    using Rows = ResidentRows<ND, KN, MORE, T, TV>;
    constexpr int kDofs = Rows::kDofs;
    Rows rows;
    char *lds = reinterpret_cast<char *>(dyn_lds);
    bool fits;
    lds += rows.setup(a, lds, sizeof(T) * ND * a.chunk, sizeof(T) * ND, fits);
    T *ps = reinterpret_cast<T *>(lds);
    T *sq = ps + size_t(rows.Hn + 1) * ND;
    const int t = threadIdx.x, nd = rows.cnt * ND;
    const int64_t d0 = ND * rows.n0;
    unsigned epoch = a.epoch;
    if (!resident_fits(a, fits, epoch)) return;
    auto gave_up = [&] {
        if (t == 0) a.host->aborted = kGaveUp;
    };
    if (t < ND) ps[rows.Hn * ND + t] = T(0);
    T x[kDofs], r[kDofs], di[kDofs];
#pragma unroll
    for (int k = 0; k < kDofs; ++k) {
        const int e = t + k * kResThreads;
        const bool own = e < nd;
        x[k] = own && a.it0 > 0 ? a.x[d0 + e] : T(0);
        r[k] = own ? (a.it0 > 0 ? a.r[d0 + e] : a.b[d0 + e]) : T(0);
        di[k] = own && !a.bj ? a.dinv[d0 + e] : T(0);
    }
    // z = M r of the owned entries, also to memory for the others; sums of r z and r r
    auto precondition = [&](double (&dots)[2]) {
        dots[0] = dots[1] = 0.0;
        if (a.bj) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kDofs; ++k)
                if (t + k * kResThreads < nd) sq[t + k * kResThreads] = r[k];
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < kDofs; ++k) {
            const int e = t + k * kResThreads;
            if (e >= nd) continue;
            T z = di[k] * r[k];
            if (a.bj) {
                const T *M = a.dinv + ND * (d0 + e), *rn = sq + e / ND * ND;
                z = M[0] * rn[0];
#pragma unroll
                for (int c = 1; c < ND; ++c) z += M[c] * rn[c];
            }
            store_agent(a.rh + d0 + e, z);
            dots[0] += double(r[k]) * double(z);
            dots[1] += double(r[k]) * double(r[k]);
        }
    };
    // p = z + beta p on all touched nodes
    auto direction = [&](bool first, T beta) {
        rows.gather(a.rh, [&](int e, T ze) { ps[e] = first ? ze : ze + beta * ps[e]; });
#pragma unroll
        for (int k = 0; k < kDofs; ++k) {
            const int e = t + k * kResThreads;
            if (e >= nd) continue;
            const T z = a.bj ? load_agent(a.rh + d0 + e) : di[k] * r[k];
            ps[e] = first ? z : z + beta * ps[e];
        }
        __syncthreads();
    };
    double rho, bnorm2, rnorm2, tol2;
    int its = a.it0, converged = 0, breakdown = 0;
    if (a.it0 == 0) {
        double dots[2], tot[2];
        precondition(dots);
        if (!grid_sum<2>(a.slots, epoch++, a.limit, dots, tot)) return gave_up();
        rho = tot[0];
        bnorm2 = rnorm2 = tot[1];
        tol2 = uniform(a.rtol * a.rtol * bnorm2);
        breakdown = isfinite(tot[1]) ? 0 : 2;
        converged = tot[1] == 0.0;
        direction(true, T(0));
    } else {
        rho = a.sc->rho;  // (rewritten by workgroup 0 after the first round only)
        bnorm2 = a.sc->bnorm2;
        rnorm2 = a.sc->rnorm2;
        tol2 = a.sc->tol2;
        for (int e = t; e < nd; e += kResThreads) ps[e] = a.p[d0 + e];
        rows.gather(a.p, [&](int e, T pe) { ps[e] = pe; });
        __syncthreads();
    }
    for (int it = a.it0; it < a.it_end && !converged && !breakdown; ++it) {
        double dot[1] = {0.0}, pq[1];
        rows.product(ps, [&](int ln, T q) {
            const int e = ln * ND + (t & 7);
            sq[e] = q;
            dot[0] += double(ps[e]) * double(q);
        });
        if (!grid_sum<1>(a.slots, epoch++, a.limit, dot, pq)) return gave_up();
        if (!(pq[0] > 0.0) || !isfinite(pq[0])) {  // CG needs (p, K p) > 0
            breakdown = 1;
            break;
        }
        const T al = T(rho / pq[0]);
#pragma unroll
        for (int k = 0; k < kDofs; ++k) {
            const int e = t + k * kResThreads;
            if (e >= nd) continue;
            x[k] += al * ps[e];
            r[k] -= al * sq[e];
        }
        double dots[2], tot[2];
        precondition(dots);
        if (!grid_sum<2>(a.slots, epoch++, a.limit, dots, tot)) return gave_up();
        its = it + 1;
        rnorm2 = tot[1];
        breakdown = uniform(!isfinite(tot[0]) || !isfinite(tot[1]) ? 2 : 0);
        converged = uniform(int(!breakdown && tot[1] <= tol2));
        const T beta = T(tot[0] / rho);
        rho = tot[0];
        if (!converged && !breakdown) direction(false, beta);
    }
#pragma unroll
    for (int k = 0; k < kDofs; ++k) {
        const int e = t + k * kResThreads;
        if (e >= nd) continue;
        a.x[d0 + e] = x[k];
        a.r[d0 + e] = r[k];
        if (!converged && !breakdown) a.p[d0 + e] = ps[e];
    }
    if (blockIdx.x == 0 && t == 0)
        for (KrylovScalars *sc : {a.sc, a.host}) {
            sc->rho = rho;
            sc->bnorm2 = bnorm2;
            sc->rnorm2 = rnorm2;
            sc->tol2 = tol2;
            sc->its = its;
            sc->converged = converged;
            sc->breakdown = breakdown;
        }
}

// BiCGSTAB on K D^{-1} (point Jacobi folded into the values), likewise.  LDS: p, r (s in its
// second half) and v on the touched nodes, rhat and t on the owned ones; v and t
// cross the chip.
template <int ND, int KN, bool MORE, typename T, typename TV>
__global__ __launch_bounds__(kResThreads, 2) void k_bicg_resident(ResidentArgs<T, TV> a) {
    extern __shared__ double dyn_lds[];
    using Rows = ResidentRows<ND, KN, MORE, T, TV>;
    constexpr int kDofs = Rows::kDofs;
    Rows rows;
    char *lds = reinterpret_cast<char *>(dyn_lds);
    bool fits;
    lds += rows.setup(a, lds, 2 * sizeof(T) * ND * a.chunk, 3 * sizeof(T) * ND, fits);
    T *ps = reinterpret_cast<T *>(lds);
    T *rs = ps + size_t(rows.Hn + 1) * ND;
    T *vs = rs + size_t(rows.Hn + 1) * ND;
    T *hs = vs + size_t(rows.Hn + 1) * ND;  // rhat
    T *ts = hs + size_t(a.chunk) * ND;
    const int t = threadIdx.x, nd = rows.cnt * ND, nh = rows.Hn * ND;
    const int64_t d0 = ND * rows.n0;
    unsigned epoch = a.epoch;
    if (!resident_fits(a, fits, epoch)) return;
    auto gave_up = [&] {
        if (t == 0) a.host->aborted = kGaveUp;
    };
    // entries of a vector written before the launch, on the touched nodes
    if (t < ND) ps[nh + t] = rs[nh + t] = T(0);
    auto load_touched = [&](const T *src, T *dst) {
        for (int e = t; e < nd; e += kResThreads) dst[e] = src[d0 + e];
        rows.gather(src, [&](int e, T se) { dst[e] = se; });
    };
    T x[kDofs];
    double rho, alpha, omega, beta, bnorm2, rnorm2, tol2, rh2, rmin2;
    int its = a.it0, converged = 0, breakdown = 0;
    bool restart = false;
    if (a.it0 == 0) {
        load_touched(a.b, rs);
        for (int e = t; e < nh; e += kResThreads) ps[e] = vs[e] = T(0);
        __syncthreads();
        double dots[1] = {0.0}, tot[1];
#pragma unroll
        for (int k = 0; k < kDofs; ++k) {
            const int e = t + k * kResThreads;
            x[k] = T(0);
            if (e >= nd) continue;
            hs[e] = rs[e];
            dots[0] += double(rs[e]) * double(rs[e]);
        }
        if (!grid_sum<1>(a.slots, epoch++, a.limit, dots, tot)) return gave_up();
        rho = bnorm2 = rnorm2 = rh2 = rmin2 = tot[0];
        tol2 = uniform(a.rtol * a.rtol * bnorm2);
        breakdown = isfinite(tot[0]) ? 0 : 2;
        converged = tot[0] == 0.0;
        alpha = omega = 1.0;
        beta = 0.0;
    } else {
        const KrylovScalars &sc = *a.sc;  // (rewritten by workgroup 0 after the first round only)
        rho = sc.rho, alpha = sc.alpha, omega = sc.omega, beta = sc.beta;
        bnorm2 = sc.bnorm2, rnorm2 = sc.rnorm2, tol2 = sc.tol2, rh2 = sc.rh2, rmin2 = sc.rmin2;
        restart = sc.restart_at == a.it0;
        load_touched(a.r, rs);
        load_touched(a.p, ps);
        load_touched(a.v, vs);
#pragma unroll
        for (int k = 0; k < kDofs; ++k) {
            const int e = t + k * kResThreads;
            x[k] = e < nd ? a.x[d0 + e] : T(0);
            if (e < nd) hs[e] = a.rh[d0 + e];
        }
        // all have read v before anyone's first product writes it
        const double none[1] = {0.0};
        double all[1];
        if (!grid_sum<1>(a.slots, epoch++, a.limit, none, all)) return gave_up();
    }
    for (int it = a.it0; it < a.it_end && !converged && !breakdown; ++it) {
        {
            const T bt = T(beta), om = T(omega);
            for (int e = t; e < nh; e += kResThreads) {
                const T re = rs[e];
                ps[e] = restart ? re : re + bt * (ps[e] - om * vs[e]);
                if (restart && e < nd) hs[e] = re;
            }
        }
        __syncthreads();
        double dot[1] = {0.0}, hv[1];
        rows.product(ps, [&](int ln, T q) {
            const int e = ln * ND + (t & 7);
            store_agent(a.v + d0 + e, q);
            vs[e] = q;
            dot[0] += double(hs[e]) * double(q);
        });
        if (!grid_sum<1>(a.slots, epoch++, a.limit, dot, hv)) return gave_up();
        if (!(hv[0] != 0.0) || !isfinite(hv[0])) {  // (rhat, v) vanished
            breakdown = 1;
            break;
        }
        alpha = uniform(rho / hv[0]);
        const T al = T(alpha);
        rows.gather(a.v, [&](int e, T ve) {
            vs[e] = ve;
            rs[e] -= al * ve;
        });
        for (int e = t; e < nd; e += kResThreads) rs[e] -= al * vs[e];
        __syncthreads();
        double sdots[3] = {0.0, 0.0, 0.0}, stot[3];  // (t, s), (t, t), (s, s)
        rows.product(rs, [&](int ln, T q) {
            const int e = ln * ND + (t & 7);
            store_agent(a.t + d0 + e, q);
            ts[e] = q;
            const double se = double(rs[e]), qe = double(q);
            sdots[0] += qe * se;
            sdots[1] += qe * qe;
            sdots[2] += se * se;
        });
        if (!grid_sum<3>(a.slots, epoch++, a.limit, sdots, stot)) return gave_up();
        omega = uniform(bicg_omega<T>(stot));
        const T om = T(omega);
        double rdots[2] = {0.0, 0.0}, rtot[2];  // (rhat, r), |r|^2
#pragma unroll
        for (int k = 0; k < kDofs; ++k) {
            const int e = t + k * kResThreads;
            if (e >= nd) continue;
            const T se = rs[e];
            x[k] += al * ps[e] + om * se;
            const T re = se - om * ts[e];
            rs[e] = re;
            rdots[0] += double(hs[e]) * double(re);
            rdots[1] += double(re) * double(re);
        }
        rows.gather(a.t, [&](int e, T te) { rs[e] -= om * te; });
        if (!grid_sum<2>(a.slots, epoch++, a.limit, rdots, rtot)) return gave_up();
        const BicgStart b = bicg_start(rtot, tol2, bnorm2, rh2, rmin2, omega, bicg_rho_floor<T>());
        its = it + 1;
        rnorm2 = b.r2;
        breakdown = uniform(b.nan ? 2 : (b.div ? 1 : 0));
        converged = uniform(int(b.conv));
        restart = uniform(int(b.restart)) != 0;
        beta = uniform(restart ? 0.0 : (b.rho / rho) * (alpha / omega));
        rho = uniform(b.rho);
        rh2 = uniform(b.rh2);
        rmin2 = uniform(b.rmin2);
    }
#pragma unroll
    for (int k = 0; k < kDofs; ++k) {
        const int e = t + k * kResThreads;
        if (e >= nd) continue;
        a.x[d0 + e] = x[k];
        if (!converged && !breakdown) {
            a.r[d0 + e] = rs[e];
            a.p[d0 + e] = ps[e];
            a.rh[d0 + e] = hs[e];
        }
    }
    if (blockIdx.x == 0 && t == 0)
        for (KrylovScalars *sc : {a.sc, a.host}) {
            sc->rho = rho, sc->alpha = alpha, sc->omega = omega, sc->beta = beta;
            sc->bnorm2 = bnorm2, sc->rnorm2 = rnorm2, sc->tol2 = tol2, sc->rh2 = rh2, sc->rmin2 = rmin2;
            sc->restart_at = restart ? its : -1;
            sc->its = its;
            sc->converged = converged;
            sc->breakdown = breakdown;
        }
}

// Workgroups of resident solves on one device wait for one another, so all of them have to
// fit the device at once: a solve takes its share of the compute units here before the
// launch and gives it back when its kernel has ended (other threads' solves wait).  Workgroups
// go to the 8 XCDs in turn, so what has to fit is what falls on the first one: with 250 + 6
// workgroups on 256 compute units two XCDs would get 33 for their 32, and each kernel could
// wait for the unit that the other holds.
class ComputeUnits {
public:
    ComputeUnits(int device, int n, int total) : pool_(pool(device)), n_(std::min((n + 7) / 8 * 8, total)) {
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
    int kn = 0, grid = 0, chunk = 0, check_fit = 0;
    int lds = 0;
};

template <int ND, typename TV>
constexpr int resident_max() { return ND == 1 || sizeof(TV) == 4 ? 4 : 2; }
// the same where other rows are read again (their blocks in flight need registers too)
template <int ND, typename TV>
constexpr int resident_max_more() { return ND == 1 ? 4 : (sizeof(TV) == 4 ? 3 : 2); }

// Nodes per 8-lane group kept in registers (kn), workgroups and LDS.  Few workgroups sum
// faster, many have shorter rows of work: the smallest kn that needs at most 80 (one dof per
// node: 40), else the largest.  Time per iteration with a limit of 16 / 80 / 256: BiCGSTAB,
// FP32 values under FP64 vectors, N = 14,739 17.1 / 12.1 / 12.3 us; 46,875 17.7 / 17.7 / 16.3;
// CG, FP64, 4,131 6.5 / 6.0 / 6.0; 26,877 7.8 / 7.8 / 8.3; CG, FP32, 26,877 7.7 / 6.9 / 7.7; one
// dof per node, 9,261 6.4 / 6.8 / 8.2 and 6.3 at 40.  At most two owned dofs per thread
// (1,024 a workgroup, so 341 nodes of three: 87,296 nodes on 256 CUs).
template <int ND, typename T, typename TV, bool CG>
ResidentPlan resident_plan(const fem_handle *h) {
    constexpr int kMax = resident_max<ND, TV>();
    const Graph &g = h->g;
    ResidentPlan p;
    if (g.max_deg < 1 || g.max_deg > kResMaxDeg) return p;
    int kn = 1;
    while (kn < kMax && g.Nn > int64_t(kn) * kResGroups * std::min(ND == 1 ? 40 : 80, h->num_cus)) kn *= 2;
    const int64_t per = int64_t(kn) * kResGroups;
    const int64_t grid = std::min<int64_t>((g.Nn + per - 1) / per, h->num_cus);
    const int64_t chunk = (g.Nn + grid - 1) / grid;
    if (chunk * ND > kResDofs * kResThreads) return p;
    // the kernels' LDS if every row touched max_deg nodes of its own
    const bool more = chunk > kMax * kResGroups;
    const int64_t W = (g.Nn + 31) / 32, touched = std::min<int64_t>(chunk * g.max_deg, g.Nn) + 1;
    const size_t need = W * (sizeof(unsigned) + sizeof(uint16_t)) + (chunk + 1 + touched) * sizeof(int) +
                        (more ? (chunk - resident_max_more<ND, TV>() * kResGroups) * g.max_deg * sizeof(uint16_t) : 0) +
                        size_t(CG ? 1 : 2) * chunk * ND * sizeof(T) + size_t(CG ? 1 : 3) * ND * sizeof(T) * touched + 16;
    const size_t room = size_t(h->lds_bytes) - kResStaticLds;
    p.check_fit = need > room;
    p.kn = kn;
    p.grid = int((g.Nn + chunk - 1) / chunk);
    p.chunk = int(chunk);
    p.lds = int(more ? room : std::min(need, room));
    return p;
}

template <int ND, int KN, bool MORE, typename T, typename TV, bool CG>
void resident_launch(const ResidentPlan &pl, const ResidentArgs<T, TV> &a, hipStream_t s) {
    void (*kernel)(ResidentArgs<T, TV>) = 
        CG ? k_cg_resident<ND, KN, MORE, T, TV> : k_bicg_resident<ND, KN, MORE, T, TV>;
    if (pl.lds > 65536)
        FEM_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, pl.lds));
    hipLaunchKernelGGL(kernel, dim3(pl.grid), dim3(kResThreads), pl.lds, s, a);
    FEM_HIP(hipGetLastError());
}

template <int ND, typename T, typename TV, bool CG>
bool resident_solve(fem_handle *h, const KrylovVecs<T> &k, const TV *values, const T *b, double rtol, int64_t max_its,
                    KrylovScalars &hs, hipStream_t s) {
    bool &misfit = h->res_misfit[CG ? 1 : 0][sizeof(T) == 8][sizeof(TV) == 8];
    if (misfit) return false;
    const ResidentPlan pl = resident_plan<ND, T, TV, CG>(h);
    if (pl.kn == 0) return false;
    if (h->res_skip > 0) {
        h->res_skip--;
        return false;
    }
    const Graph &g = h->g;
    ResidentArgs<T, TV> a{};
    a.Nn = g.Nn, a.node_ptr = g.node_ptr, a.node_nb = g.node_nb, a.values = values;
    a.b = b, a.dinv = k.dinv, a.x = k.x, a.r = k.r, a.p = k.p, a.v = k.v, a.t = k.t, a.rh = k.rh;
    a.sc = k.sc, a.host = h->host_kry, a.slots = h->res_slots;
    a.chunk = pl.chunk, a.lds = pl.lds, a.check_fit = pl.check_fit, a.bj = k.bj;
    a.rtol = rtol;
    a.limit = h->res_wait_us * h->clock_khz / 1000;
    ComputeUnits share(h->device, pl.grid, h->num_cus);
    for (;;) {
        a.it_end = int(std::min<int64_t>(max_its, int64_t(a.it0) + h->res_launch_its));
        if (h->res_epoch > 0x70000000u) {  // round numbers of the far past must not come up again
            FEM_HIP(hipMemsetAsync(h->res_slots, 0, resident_slots_bytes(h), s));
            h->res_epoch = 0;
        }
        a.epoch = h->res_epoch + 1;
        h->res_epoch += 3 * kResItsPerLaunch + 8;  // (at most two rounds before the first iteration)
        h->host_kry->aborted = 0;
        constexpr int kMax = resident_max<ND, TV>();
        if (pl.chunk > kMax * kResGroups) resident_launch<ND, resident_max_more<ND, TV>(), true, T, TV, CG>(pl, a, s);
        else if (pl.kn == 1) resident_launch<ND, 1, false, T, TV, CG>(pl, a, s);
        else if (pl.kn == 2) resident_launch<ND, 2, false, T, TV, CG>(pl, a, s);
        else resident_launch<ND, kMax, false, T, TV, CG>(pl, a, s);
        h->res_counts.launches++;
        FEM_HIP(hipStreamSynchronize(s));
        hs = *h->host_kry;
        if (hs.aborted == kGaveUp) {
            // the workgroups were not all running together (compute units held by other
            // work): the separate kernels take this solve and the next one, then, while it
            // goes on, the next 2, 4 ... 64, so that waiting in vain stays a small part
            h->res_skip = h->res_backoff;
            h->res_backoff = std::min(2 * h->res_backoff, kResMaxBackoff);
            h->res_counts.gave_up++;
            return false;
        }
        if (hs.aborted == kMisfit) {  // too many touched nodes for the LDS
            misfit = true;
            h->res_counts.misfits++;
            return false;
        }
        if (hs.converged || hs.breakdown || hs.its >= max_its) {
            h->res_counts.solves++;
            h->res_backoff = 1;
            return true;
        }
        a.it0 = hs.its;
    }
}

template <typename T, typename TV, bool CG>
bool resident_solve_nd(fem_handle *h, const KrylovVecs<T> &k, const TV *values, const T *b, double rtol,
                       int64_t max_its, KrylovScalars &hs, hipStream_t s) {
    return h->g.nd == 1 ? resident_solve<1, T, TV, CG>(h, k, values, b, rtol, max_its, hs, s)
                        : resident_solve<3, T, TV, CG>(h, k, values, b, rtol, max_its, hs, s);
}

}  // namespace

size_t resident_slots_bytes(const fem_handle *h) {
    return size_t(4) * kSlotWords * h->num_cus * sizeof(unsigned long long);
}

template <typename T>
bool kry_resident(fem_handle *h, const KrylovVecs<T> &k, bool cg, const T *b, double rtol, int64_t max_its,
                  KrylovScalars &hs, hipStream_t s) {
    if (k.layout != LAYOUT_CSR || h->g.N == 0 || (!cg && !k.fold)) return false;
    if constexpr (sizeof(T) == 8) {
        if (k.A32)
            return cg ? resident_solve_nd<T, float, true>(h, k, k.A32, b, rtol, max_its, hs, s)
                      : resident_solve_nd<T, float, false>(h, k, k.A32, b, rtol, max_its, hs, s);
    }
    return cg ? resident_solve_nd<T, T, true>(h, k, k.A, b, rtol, max_its, hs, s)
              : resident_solve_nd<T, T, false>(h, k, k.A, b, rtol, max_its, hs, s);
}

template bool kry_resident<float>(fem_handle *, const KrylovVecs<float> &, bool, const float *, double, int64_t,
                                  KrylovScalars &, hipStream_t);
template bool kry_resident<double>(fem_handle *, const KrylovVecs<double> &, bool, const double *, double, int64_t,
                                   KrylovScalars &, hipStream_t);

}  // namespace fem
