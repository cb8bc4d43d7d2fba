// Sparse matrix-vector products and Jacobi-preconditioned Krylov kernels.
//
// The CSR matrix is stored over all dofs with node-major interleaved components, so
// the ND rows of node n are contiguous and each of them lists the node's neighbour
// blocks in the same order.  The SpMV therefore walks the node graph (one 32-bit
// column index per ND x ND block) instead of the scalar column array: a group of 32
// lanes owns one node, lane l takes the l-th neighbour block, and the ND row sums
// are finished with a 32-lane reduction built from cross-lane register moves.
//
// Krylov inner products are FP64 and deterministic: every block stores its partial
// sum (fixed lane order), and the next kernel sums the partials in block order,
// either in a one-block finalize kernel or redundantly in every block of the next
// vector kernel (CG).  Scalars of the method live on the device; the host only reads
// the convergence flag every few iterations.
//
// Paper: BiCGSTAB with a Jacobi preconditioner is the linear solver inside Newton
// (Sec. 5, item 2; van der Vorst 1992).
#include <algorithm>
#include <type_traits>

#include "bicg_rules.h"
#include "internal.h"
#include "lanes.h"

namespace fem {

namespace {

constexpr int kThreads = 256;

inline unsigned grid_for(int64_t n, int threads) { return unsigned((n + threads - 1) / threads); }

template <int G, typename T>
__device__ __forceinline__ T group_sum(T v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, G);
    return v;
}

// y = alpha K^T x + beta y.  A 32-lane group takes one node, lane = neighbour block: block
// (n, m) of K^T is the transpose of block (m, n), whose place in node m's rows `mirror`
// gives.  Four dependent loads per block (row start of n, neighbour and mirror, row start of
// m, values and x) with nothing to reuse, so what counts is how many are in flight: every
// lane handles one block, eight wavefronts per SIMD, and the group's sums end in a
// reduce-scatter.  41x33x27 (9.6 M entries), against 16 lanes with two blocks each in a row:
// FP64 35.7 -> 22.9 us where the matrix is still in the Infinity Cache from the product before,
// 10% less on one that is not (ten matrices in turn, 8 us of event timing included: FP64
// 43.5 -> 39.0 us, FP32 37.5 -> 28.7).
template <int ND, typename T>
__global__ __launch_bounds__(kThreads, 8) void k_spmv_t(int64_t Nn, const int64_t *__restrict__ node_ptr,
                                                        const int32_t *__restrict__ node_nb,
                                                        const int32_t *__restrict__ mirror,
                                                        const T *__restrict__ values, const T *__restrict__ x,
                                                        T *__restrict__ y, T alpha, T beta) {
    constexpr int G = 32;
    const int lane = threadIdx.x % G;
    // blocks of one XCD take adjacent nodes: a cache line of node m's rows serves its neighbours
    const int64_t blk = int64_t(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const int64_t n = blk * (kThreads / G) + threadIdx.x / G;
    const bool live = n < Nn;  // (every lane stays active for the reduction)
    const int64_t b0 = live ? node_ptr[n] : 0;
    const int deg = live ? int(node_ptr[n + 1] - b0) : 0;
    T acc[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) acc[i] = T(0);
    for (int l = lane; l < deg; l += G) {
        const int64_t m = node_nb[b0 + l], kb = mirror[b0 + l];
        const int64_t mb0 = node_ptr[m];
        const int64_t row = int64_t(ND) * (node_ptr[m + 1] - mb0);
        const T *mv = values + int64_t(ND) * ND * mb0 + ND * (kb - mb0);
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const T xk = x[ND * m + k];
#pragma unroll
            for (int i = 0; i < ND; ++i) acc[i] += mv[k * row + i] * xk;
        }
    }
    T sv;
    if constexpr (ND == 3) sv = group32_sum3(acc[0], acc[1], acc[2], lane);
    else sv = group32_sum(acc[0], lane);
    // lanes 0, 8, 16 hold rows 0, 1, 2 of the node
    if (live && (lane & 7) == 0 && lane < 8 * ND) {
        const int64_t d = ND * n + lane / 8;
        T out = alpha * sv;
        if (beta != T(0)) out += beta * y[d];
        y[d] = out;
    }
}

// ------------------------------------------------------------------ deterministic reductions
// Grid-wide FP64 sums are done in two kernels: every block of the producing kernel
// stores its block total to partials[c * G + blockIdx.x] (plain stores, no fences or
// atomics: on a multi-XCD device a device-scope fence per block would write back the
// XCD's L2 every time), and a one-block finalize kernel launched next on the same
// stream adds the G partials in block order.  The result is bit-reproducible.
template <int NV>
__device__ void block_store_partials(const double v[NV], double *partials) {
    __shared__ double red[kThreads / 64][NV];
    const int wave = threadIdx.x / 64;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const double t = wave_sum(v[c]);
        if ((threadIdx.x & 63) == 0) red[wave][c] = t;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kThreads / 64; ++k) t += red[k][threadIdx.x];
        partials[threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// Totals of the G partials of each of NV sums, in every thread of the block.
template <int NV>
__device__ void sum_partials(const double *partials, int G, double tot[NV]) {
    __shared__ double red[kThreads / 64][NV];
    const int wave = threadIdx.x / 64;
    double v[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) v[c] = 0.0;
    for (int b = threadIdx.x; b < G; b += kThreads)
#pragma unroll
        for (int c = 0; c < NV; ++c) v[c] += partials[c * G + b];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const double t = wave_sum(v[c]);
        if ((threadIdx.x & 63) == 0) red[wave][c] = t;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kThreads / 64; ++k) t += red[k][c];
        tot[c] = t;
    }
}

// Contiguous node range of this block.  Blocks are dealt round-robin to the 8 XCDs,
// so the logical block index groups the blocks of one XCD onto adjacent ranges and
// each XCD's L2 sees a compact slab of the mesh (the x-vector gathers stay local).
__device__ __forceinline__ void block_range(int64_t Nn, int64_t &n0, int64_t &n1) {
    const unsigned G = gridDim.x, b = blockIdx.x;
    const unsigned per = G / 8;
    unsigned L = (G % 8 == 0) ? (b % 8) * per + b / 8 : b;
    int64_t chunk = (Nn + G - 1) / G;
    n0 = int64_t(L) * chunk;
    n1 = n0 + chunk < Nn ? n0 + chunk : Nn;
}

__device__ __forceinline__ bool stopped(const KrylovScalars *sc) { return sc->converged | sc->breakdown; }

// ------------------------------------------------------------------ Krylov scalars
// The scalar updates of the fused CG and BiCGSTAB iterations.  Every block of the kernel
// that needs them sums the previous kernel's partials itself, in the same order, so all
// blocks agree bit for bit; block 0 publishes the scalars.  They return false when the
// iteration stops here (converged or broken down).

// CG after iteration it: rho = (r, z), |r|^2; convergence test; beta = rho / rho_pp[it & 1].
__device__ bool cg_p_scalars(const double *partials, int count, KrylovScalars *sc, int it, double &beta) {
    double tot[2];
    sum_partials<2>(partials, count, tot);
    const double rho_prev = sc->rho_pp[it & 1];
    const bool nan = !isfinite(tot[0]) || !isfinite(tot[1]);
    const bool conv = !nan && tot[1] <= sc->tol2;
    beta = tot[0] / rho_prev;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->rho_old = rho_prev;
        sc->rho = tot[0];
        sc->rho_pp[(it + 1) & 1] = tot[0];
        sc->beta = beta;
        sc->rnorm2 = tot[1];
        sc->its = it + 1;
        if (nan) sc->breakdown = 2;
        else if (conv) sc->converged = 1;
    }
    return !(nan || conv);
}

// Tests at the start of iteration i (>= 1), with the scalars of iteration i - 1.
__device__ __forceinline__ BicgStart bicg_start_at(const double tot[2], const KrylovScalars *sc, int i,
                                                   double rho_floor) {
    const int q = (i - 1) & 1;
    return bicg_start(tot, sc->tol2, sc->bnorm2, sc->rh2_pp[q], sc->rmin2_pp[q], sc->omega_pp[q], rho_floor);
}

__device__ __forceinline__ void bicg_publish_start(const BicgStart &b, KrylovScalars *sc, int i) {
    sc->its = i;
    sc->rnorm2 = b.r2;
    if (b.nan) sc->breakdown = 2;
    else if (b.conv) sc->converged = 1;
    else if (b.div) sc->breakdown = 1;
}

// BiCGSTAB at the start of iteration it: p = r + beta (p - omega v), or p = r on a restart.
template <typename T>
__device__ bool bicg_p_scalars(const double *partials, int count, KrylovScalars *sc, int it, double &beta,
                               double &omega, bool &restart) {
    restart = false;
    beta = omega = 0.0;
    if (it == 0) return true;
    double tot[2];
    sum_partials<2>(partials, count, tot);
    const BicgStart b = bicg_start_at(tot, sc, it, bicg_rho_floor<T>());
    const int q = (it - 1) & 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        bicg_publish_start(b, sc, it);
        sc->rho_old = sc->rho_pp[q];
        sc->rho = b.rho;
        sc->rho_pp[it & 1] = b.rho;
        sc->rh2_pp[it & 1] = b.rh2;
        sc->rmin2_pp[it & 1] = b.rmin2;
        if (b.restart) sc->restart_at = it;
    }
    if (b.nan || b.conv || b.div) return false;
    restart = b.restart;
    omega = sc->omega_pp[q];
    if (!restart) beta = (b.rho / sc->rho_pp[q]) * (sc->alpha_pp[q] / omega);
    return true;
}

// BiCGSTAB in iteration it: alpha = rho_it / (rhat, v), s = r - alpha v.
__device__ bool bicg_s_scalars(const double *partials, int count, KrylovScalars *sc, int it, double &alpha) {
    double tot[1];
    sum_partials<1>(partials, count, tot);
    if (!(tot[0] != 0.0) || !isfinite(tot[0])) {  // (rhat, v) vanished
        if (blockIdx.x == 0 && threadIdx.x == 0) sc->breakdown = 1;
        return false;
    }
    alpha = sc->rho_pp[it & 1] / tot[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->alpha_pp[it & 1] = alpha;
        sc->alpha = alpha;
    }
    return true;
}

// How k_spmv_nodes gets its input vector: read it (GATHER_X), or form it from the
// iteration's vectors while gathering, which saves the vector kernel that would write it
// first.  The block writes its own rows of the formed vector to `out`.
//   GATHER_CG_P:   p = z + beta p_old                      x = z, b = p_old
//   GATHER_BICG_P: p = r + beta (p_old - omega v_old)      x = r, b = p_old, c = v_old
//                  (on a restart p = r, and rh = r)
//   GATHER_BICG_S: s = r - alpha v                         x = r, b = v
enum { GATHER_X = 0, GATHER_CG_P = 1, GATHER_BICG_P = 2, GATHER_BICG_S = 3 };
template <typename T>
struct GatherIn {
    const T *b = nullptr, *c = nullptr;
    T *out = nullptr, *rh = nullptr;
    const double *partials = nullptr;  // of the kernel before (count of them)
    int count = 0, it = 0;
};

// Persistent SpMV over this block's contiguous node range.  The range's row
// pointers are staged in LDS once; each 32-lane group then takes one node at a time,
// and the next node's index and value loads are issued before the current x gathers
// are awaited.  Lane l of a group handles neighbour block l of its node (node degrees
// above 32 fall back to a strided loop); the ND row sums are finished with a
// reduce-scatter over the group (a row swap and four DPP steps, no LDS traffic).
// Row results are kept in LDS and written (with the dot-product terms) after the
// chunk.  D16: column blocks read as 16-bit offsets from the row node (half the index
// bytes) when the node numbering allows it.
//
// MODE 0: y = alpha K x + beta y
// MODE 1: y = K x and alpha = rho / (w0, y)                 (BiCGSTAB v = K ph, CG q = K p)
// MODE 2: y = K x and omega = (w0, y) / (y, y), w0 = s      (BiCGSTAB t = K sh)
//
// What bounds it: bytes from HBM, or from the 256 MB Infinity Cache when the matrix
// fits there.  The values are read with ordinary (cached) loads: non-temporal ones kept small
// matrices out of the Infinity Cache, and a lane's 12- or 24-byte pieces and the rows of
// neighbouring nodes share cache lines.  One node in flight per group and few resident
// blocks (spmv_grid).  The gain is not one of traffic: beyond L2 the 100^3 product moves 1.31
// instead of 1.19 GB with FP32 values under FP64 vectors, 1.18 instead of 1.15 with FP32 vectors and
// 2.25 instead of 2.28 in FP64, at a higher rate (4.50 -> 5.89 TB/s of algorithmic bytes in
// FP64).  Back-to-back products on box meshes, non-temporal loads with 4 / 4 / 2 nodes
// in flight on every resident block against this form:
//   FP64, 100^3 (2.08 GB)     461.8 -> 352.2 us (4.50 -> 5.89 TB/s)
//   FP64, 64x32x32 (138 MB)    36.8 ->  22.4 us (3.76 -> 6.17 TB/s)
//   FP64, 24x24x48 (59 MB)     17.7 ->  11.2 us
//   FP32, 100^3 (1.07 GB)     202.9 -> 183.6 us (5.27 -> 5.82 TB/s)
//   FP32, 64^3 (282 MB)        57.8 ->  44.4 us
//   FP32 values under FP64 vectors, 100^3   221.5 -> 203.8 us; 40^3  17.3 -> 13.2 us
//   one dof per node, FP64, 50x50x10         7.6 ->   4.8 us
// (a plain read of the same values takes 325, 20, 7.4-8.5, 176, 41 us).
constexpr int kSpmvGroup = 32;
constexpr int kMaxChunk = 1024;  // nodes per block staged in LDS

template <int ND, int MODE, typename T, bool D16, typename TV = T, int GATHER = GATHER_X>
__global__ __launch_bounds__(kThreads, 4) void k_spmv_nodes(int64_t Nn, const int64_t *__restrict__ node_ptr,
                                                            const int32_t *__restrict__ node_nb,
                                                            const int16_t *__restrict__ node_dnb,
                                                            const TV *__restrict__ values, const T *__restrict__ x,
                                                            T *__restrict__ y, const T *__restrict__ w0, T alpha,
                                                            T beta, double *partials, KrylovScalars *sc, int cg,
                                                            int big, GatherIn<T> gi = GatherIn<T>()) {
    constexpr int G = kSpmvGroup;
    constexpr int GPB = kThreads / G;  // groups per block
    static_assert(G == 32 && (ND == 1 || ND == 3), "32-lane groups, 1 or 3 dofs per node");
    __shared__ int64_t sptr[kMaxChunk + 1];
    __shared__ T sy[kMaxChunk * ND];  // the chunk's results, written out at its end
    constexpr int NDOT = MODE == 2 ? 3 : MODE;  // (w0, y); MODE 2 also (y, y) and (w0, w0)
    __shared__ double sdot[MODE != 0 ? NDOT * kThreads : 1];  // per-thread dot terms (no registers in the node loop)
    if ((MODE != 0 || sc != nullptr) && stopped(sc)) return;  // MODE 0 with sc: inside a Krylov loop
    if (MODE != 0)
        for (int c = 0; c < NDOT; ++c) sdot[c * kThreads + threadIdx.x] = 0.0;
    T c1 = T(0), c2 = T(0);
    bool restart = false;
    if constexpr (GATHER == GATHER_CG_P) {
        double beta1 = 0.0;
        if (gi.it > 0 && !cg_p_scalars(gi.partials, gi.count, sc, gi.it - 1, beta1)) return;
        c1 = T(beta1);
    } else if constexpr (GATHER == GATHER_BICG_P) {
        double beta1, omega;
        if (!bicg_p_scalars<T>(gi.partials, gi.count, sc, gi.it, beta1, omega, restart)) return;
        c1 = T(beta1);
        c2 = T(omega);
    } else if constexpr (GATHER == GATHER_BICG_S) {
        double alpha1;
        if (!bicg_s_scalars(gi.partials, gi.count, sc, gi.it, alpha1)) return;
        c1 = T(alpha1);
    }
    auto input = [&](int64_t d) -> T {
        const T a = x[d];
        if constexpr (GATHER == GATHER_CG_P) return a + c1 * gi.b[d];
        else if constexpr (GATHER == GATHER_BICG_P) return restart ? a : a + c1 * (gi.b[d] - c2 * gi.c[d]);
        else if constexpr (GATHER == GATHER_BICG_S) return a - c1 * gi.b[d];
        else return a;
    };
    int64_t r0, r1;
    block_range(Nn, r0, r1);
    const int lane = threadIdx.x % G;
    const int grp = threadIdx.x / G;
    // after the group reduction, lanes 0, 8, 16 hold rows 0, 1, 2 of the node
    const int row = (lane & 7) == 0 && lane < 8 * ND ? lane / 8 : -1;
    for (int64_t n0 = r0; n0 < r1; n0 += kMaxChunk) {
        const int cnt = int(r1 - n0 < kMaxChunk ? r1 - n0 : kMaxChunk);
        __syncthreads();  // previous sub-chunk finished with sptr
        for (int i = threadIdx.x; i <= cnt; i += kThreads) sptr[i] = node_ptr[n0 + i];
        __syncthreads();
        int deg;
        int32_t m;
        TV v[ND][ND];
        // Column index and values of one node.  Addresses are clamped (a node past the
        // chunk re-reads its last node, a lane past the degree reads block 0), so the
        // loads are branch-free; the results of such slots are masked.
        auto load_node = [&](int ln) {
            ln = ln < cnt ? ln : cnt - 1;
            const int64_t b0 = sptr[ln];
            deg = int(sptr[ln + 1] - b0);
            const int lc = lane < deg ? lane : 0;
            if constexpr (D16) m = int32_t(n0 + ln) + int32_t(node_dnb[b0 + lc]);
            else m = node_nb[b0 + lc];
            const TV *vb = values + int64_t(ND) * ND * b0 + ND * lc;
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int k = 0; k < ND; ++k) v[i][k] = vb[int64_t(i) * ND * deg + k];
        };
        load_node(grp);
        for (int ln = grp; ln < cnt; ln += GPB) {
            // Software pipeline: the x gathers of this node go out first, then the next
            // node's index and value loads, so waiting for the gathers leaves the next
            // node in flight (memory counters complete in issue order).
            T xm[ND];
            TV cv[ND][ND];
#pragma unroll
            for (int k = 0; k < ND; ++k) xm[k] = input(int64_t(ND) * m + k);
            const int cdeg = deg;
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int k = 0; k < ND; ++k) cv[i][k] = v[i][k];
            load_node(ln + GPB);
            T acc[ND];
#pragma unroll
            for (int i = 0; i < ND; ++i) {
                T a = T(0);
#pragma unroll
                for (int k = 0; k < ND; ++k) a += T(cv[i][k]) * xm[k];
                acc[i] = lane < cdeg ? a : T(0);
            }
            T sv;
            if constexpr (ND == 3) sv = group32_sum3(acc[0], acc[1], acc[2], lane);
            else sv = group32_sum(acc[0], lane);
            if (row >= 0) sy[ND * ln + row] = sv;
        }
        __syncthreads();
        if (big) {  // neighbours beyond the 32nd of high-degree nodes (none on structured meshes)
            for (int ln = grp; ln < cnt; ln += GPB) {
                const int64_t b = sptr[ln];
                const int dg = int(sptr[ln + 1] - b);
                if (dg <= G) continue;
                T acc[ND];
#pragma unroll
                for (int i = 0; i < ND; ++i) acc[i] = T(0);
                for (int l = lane + G; l < dg; l += G) {
                    const int64_t mm = node_nb[b + l];
                    const TV *vb = values + int64_t(ND) * ND * b + ND * l;
#pragma unroll
                    for (int i = 0; i < ND; ++i)
#pragma unroll
                        for (int k = 0; k < ND; ++k) acc[i] += T(vb[int64_t(i) * ND * dg + k]) * input(ND * mm + k);
                }
                T sv;
                if constexpr (ND == 3) sv = group32_sum3(acc[0], acc[1], acc[2], lane);
                else sv = group32_sum(acc[0], lane);
                if (row >= 0) sy[ND * ln + row] += sv;
            }
            __syncthreads();
        }
        // The chunk's rows go out as one coalesced pass.  Stores share the vector
        // memory counter with loads here, so a store inside the node loop would make
        // every later wait for a load also wait for that store's acknowledgement.
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
        // (non-temporal stores: measured 4% faster than cached ones for this pass)
        for (int i = threadIdx.x; i < ND * cnt; i += kThreads) {
            const int64_t d = int64_t(ND) * n0 + i;
            const T sv = sy[i];
            if (MODE == 0) {
                T out = alpha * sv;
                if (beta != T(0)) out += beta * y[d];
                __builtin_nontemporal_store(out, y + d);
            } else {
                T w;
                if constexpr (GATHER == GATHER_X) {
                    __builtin_nontemporal_store(sv, y + d);
                    w = w0[d];
                } else {  // these vectors are small and gathered again next: keep them cached
                    y[d] = sv;
                    w = input(d);
                    gi.out[d] = w;
                    if constexpr (GATHER == GATHER_BICG_P) {
                        if (restart) gi.rh[d] = w;  // p = r = rhat
                        else w = gi.rh[d];
                    }
                }
                const double wd = double(w);
                d0 += wd * double(sv);
                if (MODE == 2) {
                    d1 += double(sv) * double(sv);
                    d2 += wd * wd;
                }
            }
        }
        if (MODE != 0) {
            sdot[threadIdx.x] += d0;
            if (MODE == 2) {
                sdot[kThreads + threadIdx.x] += d1;
                sdot[2 * kThreads + threadIdx.x] += d2;
            }
        }
    }
    if constexpr (MODE != 0) {
        double vv[NDOT];
        for (int c = 0; c < NDOT; ++c) vv[c] = sdot[c * kThreads + threadIdx.x];
        block_store_partials<NDOT>(vv, partials);
    }
}

// SpMV on the symmetric block layout (blocks (n, m) with m >= n stored, block-major).
// Node n's row needs its upper blocks, which are contiguous from up_base[n], and its
// lower blocks (n, m), m < n, which are the transposes of the stored blocks (m, n)
// (index lo_val).  Those were streamed moments earlier by the block range holding
// node m, so they come from L2 or the Infinity Cache; HBM traffic is the stored half
// of the matrix.  Same persistent scheme as k_spmv_nodes (LDS-staged row data, P
// nodes in flight per 32-lane group, branch-free loads on clamped addresses).
template <int ND, int P, int MODE, typename T>
__global__ __launch_bounds__(kThreads) void k_spmv_sym(int64_t Nn, const int64_t *__restrict__ node_ptr,
                                                       const int64_t *__restrict__ up_base,
                                                       const int32_t *__restrict__ node_nb,
                                                       const int32_t *__restrict__ lo_val,
                                                       const T *__restrict__ values, const T *__restrict__ x,
                                                       T *__restrict__ y, const T *__restrict__ w0, T alpha, T beta,
                                                       double *partials, KrylovScalars *sc, int cg) {
    constexpr int G = kSpmvGroup;
    constexpr int GPB = kThreads / G;
    constexpr int CH = kMaxChunk / 2;
    constexpr int BS = ND * ND;
    __shared__ int64_t sptr[CH + 1];
    __shared__ int64_t sup[CH + 1];
    if (MODE != 0 && stopped(sc)) return;
    int64_t r0, r1;
    block_range(Nn, r0, r1);
    const int lane = threadIdx.x % G;
    const int grp = threadIdx.x / G;
    double d0 = 0.0, d1 = 0.0, d2 = 0.0;
    for (int64_t n0 = r0; n0 < r1; n0 += CH) {
        const int cnt = int(r1 - n0 < CH ? r1 - n0 : CH);
        __syncthreads();
        for (int i = threadIdx.x; i <= cnt; i += kThreads) {
            sptr[i] = node_ptr[n0 + i];
            sup[i] = up_base[n0 + i];
        }
        __syncthreads();
        for (int base = grp; base < cnt; base += P * GPB) {
            int64_t b0[P], ub[P];
            int deg[P], dpos[P];
            int32_t m[P];
            T v[P][BS];
            T xm[P][ND];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int ln = base + p * GPB;
                const bool ok = ln < cnt;
                b0[p] = ok ? sptr[ln] : 0;
                deg[p] = ok ? int(sptr[ln + 1] - sptr[ln]) : 0;
                ub[p] = ok ? sup[ln] : 0;
                dpos[p] = ok ? deg[p] - int(sup[ln + 1] - sup[ln]) : 0;
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const bool act = lane < deg[p];
                const bool lower = lane < dpos[p];
                m[p] = __builtin_nontemporal_load(node_nb + b0[p] + (act ? lane : 0));
                const int32_t lv = __builtin_nontemporal_load(lo_val + b0[p] + (lower ? lane : 0));
                const int64_t ku = lower ? int64_t(lv) : (act ? ub[p] + (lane - dpos[p]) : ub[p]);
                const T *vb = values + BS * ku;
#pragma unroll
                for (int q = 0; q < BS; ++q) v[p][q] = vb[q];
            }
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int k = 0; k < ND; ++k) xm[p][k] = x[int64_t(ND) * m[p] + k];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const bool act = lane < deg[p];
                const bool lower = lane < dpos[p];
                T acc[ND];
#pragma unroll
                for (int i = 0; i < ND; ++i) {
                    T a = T(0);
#pragma unroll
                    for (int k = 0; k < ND; ++k) a += (lower ? v[p][k * ND + i] : v[p][i * ND + k]) * xm[p][k];
                    acc[i] = act ? a : T(0);
                }
                for (int l = lane + G; l < deg[p]; l += G) {  // high-degree nodes
                    const int64_t mm = node_nb[b0[p] + l];
                    const bool lw = l < dpos[p];
                    const int64_t kk = lw ? int64_t(lo_val[b0[p] + l]) : ub[p] + (l - dpos[p]);
                    const T *vb = values + BS * kk;
#pragma unroll
                    for (int i = 0; i < ND; ++i)
#pragma unroll
                        for (int k = 0; k < ND; ++k) acc[i] += (lw ? vb[k * ND + i] : vb[i * ND + k]) * x[ND * mm + k];
                }
#pragma unroll
                for (int i = 0; i < ND; ++i) acc[i] = group_sum<G>(acc[i]);
                const int ln = base + p * GPB;
                if (ln < cnt && lane < ND) {
                    T sv = acc[0];
#pragma unroll
                    for (int i = 1; i < ND; ++i)
                        if (lane == i) sv = acc[i];
                    const int64_t d = int64_t(ND) * (n0 + ln) + lane;
                    if (MODE == 0) {
                        T out = alpha * sv;
                        if (beta != T(0)) out += beta * y[d];
                        y[d] = out;
                    } else {
                        y[d] = sv;
                        const double wd = double(w0[d]);
                        d0 += wd * double(sv);
                        if (MODE == 2) {
                            d1 += double(sv) * double(sv);
                            d2 += wd * wd;
                        }
                    }
                }
            }
        }
    }
    if constexpr (MODE != 0) {
        constexpr int NDOT = MODE == 2 ? 3 : MODE;
        double vv[3] = {d0, d1, d2};
        block_store_partials<NDOT>(vv, partials);
    }
}

// alpha = rho / (w0, y)
__global__ __launch_bounds__(kThreads) void k_fin_alpha(int G, const double *__restrict__ partials,
                                                        KrylovScalars *sc, int cg) {
    if (stopped(sc)) return;
    double tot[1];
    sum_partials<1>(partials, G, tot);
    if (threadIdx.x == 0) {
        bool bad = !(tot[0] != 0.0) || !isfinite(tot[0]) || (cg && !(tot[0] > 0.0));
        if (bad) sc->breakdown = 1;
        else sc->alpha = sc->rho / tot[0];
    }
}

// omega = (t, s) / (t, t)
__global__ __launch_bounds__(kThreads) void k_fin_omega(int G, const double *__restrict__ partials,
                                                        KrylovScalars *sc) {
    if (stopped(sc)) return;
    double tot[2];
    sum_partials<2>(partials, G, tot);
    if (threadIdx.x == 0) sc->omega = (tot[1] > 0.0 && isfinite(tot[1])) ? tot[0] / tot[1] : 0.0;
}

// BiCGSTAB (block Jacobi form): x += alpha ph + omega sh; r = s - omega t; rho_new = (rh, r); |r|^2
template <typename T>
__global__ __launch_bounds__(kThreads) void k_bicg_xr(int64_t N, T *__restrict__ x, T *__restrict__ r,
                                                      const T *__restrict__ rh, const T *__restrict__ ph,
                                                      const T *__restrict__ s, const T *__restrict__ sh,
                                                      const T *__restrict__ t, double *partials, KrylovScalars *sc) {
    if (stopped(sc)) return;
    const T al = T(sc->alpha), om = T(sc->omega);
    double d0 = 0.0, d1 = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x; i < N; i += int64_t(gridDim.x) * kThreads) {
        x[i] += al * ph[i] + om * sh[i];
        T ri = s[i] - om * t[i];
        r[i] = ri;
        d0 += double(rh[i]) * double(ri);
        d1 += double(ri) * double(ri);
    }
    double v[2] = {d0, d1};
    block_store_partials<2>(v, partials);
}

// BiCGSTAB: rho_new = (rhat, r), |r|^2; convergence, divergence and restart tests
__global__ __launch_bounds__(kThreads) void k_fin_bicg_xr(int G, const double *__restrict__ partials,
                                                          KrylovScalars *sc) {
    if (stopped(sc)) return;
    double tot[2];
    sum_partials<2>(partials, G, tot);
    if (threadIdx.x == 0) {
        sc->rho_old = sc->rho;
        sc->rho = tot[0];
        sc->rnorm2 = tot[1];
        sc->its += 1;
        if (!isfinite(tot[0]) || !isfinite(tot[1])) {
            sc->breakdown = 2;
        } else if (tot[1] <= sc->tol2) {
            sc->converged = 1;
        } else if (tot[1] > 1e12 * sc->bnorm2) {
            sc->breakdown = 1;  // diverged
        } else if (!(fabs(tot[0]) > 1e-9 * sqrt(sc->rh2 * tot[1])) || sc->omega == 0.0 ||
                   tot[1] > 1e6 * sc->rmin2) {
            // (rhat, r) lost its size relative to |rhat||r|, omega vanished, or the
            // residual grew 1000x above its best value: restart from the current r
            sc->restart_at = sc->its;
            sc->rho = tot[1];
            sc->rh2 = tot[1];
        }
        sc->rmin2 = fmin(sc->rmin2, tot[1]);
    }
}

// CG with the scalar updates folded into the vector kernels.  Each block sums the
// previous kernel's per-block partials itself (same order in every block, so all
// blocks agree bit for bit), which removes the one-block finalize launches.
//
// Iteration it: alpha = rho_pp[it & 1] / (p, q) with q = K p from the SpMV partials;
// x += alpha p; r -= alpha q; z = Dinv r; partials of (r, z) and |r|^2.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_cg_xr_fused(int64_t N, T *__restrict__ x, T *__restrict__ r,
                                                          T *__restrict__ z, const T *__restrict__ p,
                                                          const T *__restrict__ q, const T *__restrict__ dinv,
                                                          const double *__restrict__ pq_partials, int pq_count,
                                                          double *partials, KrylovScalars *sc, int it) {
    // 16-byte accesses over the bulk (the vectors are 256-byte aligned), scalar tail; the
    // first ones go out before the partials are waited for
    using V = Vec16<T>;
    constexpr int W = V::W;
    const int64_t NV = N / W, stride = int64_t(gridDim.x) * kThreads;
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    typename V::type xv{}, pv{}, rv{}, qv{}, dv{};
    auto load = [&] {
        xv = V::ld(x, i);
        pv = V::ld(p, i);
        rv = V::ld(r, i);
        qv = V::ld(q, i);
        dv = V::ld(dinv, i);
    };
    if (i < NV) load();
    if (stopped(sc)) return;
    double pq[1];
    sum_partials<1>(pq_partials, pq_count, pq);
    if (!(pq[0] > 0.0) || !isfinite(pq[0])) {  // CG needs (p, K p) > 0
        if (blockIdx.x == 0 && threadIdx.x == 0) sc->breakdown = 1;
        return;
    }
    const double alpha = sc->rho_pp[it & 1] / pq[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->alpha = alpha;
    const T al = T(alpha);
    double d0 = 0.0, d1 = 0.0;
    auto update = [&](int64_t i) {
        x[i] += al * p[i];
        T ri = r[i] - al * q[i];
        r[i] = ri;
        T zi = dinv[i] * ri;
        z[i] = zi;
        d0 += double(ri) * double(zi);
        d1 += double(ri) * double(ri);
    };
    while (i < NV) {
        xv += al * pv;
        rv -= al * qv;
        const typename V::type zv = dv * rv;
        V::st_nt(x, i, xv);
        V::st_nt(r, i, rv);
        V::st_nt(z, i, zv);
#pragma unroll
        for (int c = 0; c < W; ++c) {
            d0 += double(rv[c]) * double(zv[c]);
            d1 += double(rv[c]) * double(rv[c]);
        }
        i += stride;
        if (i < NV) load();
    }
    if (blockIdx.x == 0)
        for (int64_t i = NV * W + threadIdx.x; i < N; i += kThreads) update(i);
    double v[2] = {d0, d1};
    block_store_partials<2>(v, partials);
}

// rho = (r, z), |r|^2 from the partials; convergence test; beta = rho / rho_pp[it & 1];
// p = z + beta p.  Block 0 publishes the scalars (the new rho to the other slot).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_cg_p_fused(int64_t N, const T *__restrict__ z, T *__restrict__ p,
                                                         const double *__restrict__ rz_partials, int rz_count,
                                                         KrylovScalars *sc, int it) {
    using V = Vec16<T>;
    constexpr int W = V::W;
    const int64_t NV = N / W, stride = int64_t(gridDim.x) * kThreads;
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    typename V::type zv{}, pv{};
    auto load = [&] {
        zv = V::ld(z, i);
        pv = V::ld(p, i);
    };
    if (i < NV) load();
    if (stopped(sc)) return;
    double beta;
    if (!cg_p_scalars(rz_partials, rz_count, sc, it, beta)) return;
    const T bt = T(beta);
    while (i < NV) {
        V::st_nt(p, i, zv + bt * pv);
        i += stride;
        if (i < NV) load();
    }
    if (blockIdx.x == 0)
        for (int64_t i = NV * W + threadIdx.x; i < N; i += kThreads) p[i] = z[i] + bt * p[i];
}

// ------------------------------------------------------------------ fused BiCGSTAB
// The point-Jacobi BiCGSTAB with its scalar updates folded into the vector kernels
// (every block sums the previous kernel's partials in block order, so all blocks agree
// bit for bit and no one-block finalize kernel is launched).  Iteration i:
//   p-kernel:  rho_i, |r_i|^2 from the (rhat, r), (r, r) partials of iteration i - 1;
//              convergence, divergence and restart tests; p = r + beta (p - omega v)
//              (or p = r, rhat = r on a restart); ph = Dinv p
//   SpMV:      v = K ph with the (rhat, v) partials
//   s-kernel:  alpha = rho_i / (rhat, v); s = r - alpha v; sh = Dinv s
//   SpMV:      t = K sh with the (t, s), (t, t) partials
//   xr-kernel: omega = (t, s) / (t, t); x += alpha ph + omega sh; r = s - omega t, and
//              the (rhat, r), (r, r) partials for iteration i + 1.
// The scalars of iteration i go to slot i & 1 (see KrylovScalars).

// FOLD: the point-Jacobi scaling sits in the stored operator (K D^{-1}, see
// k_scale_columns), so the SpMV inputs are p and s themselves and ph, sh are not written.
template <typename T, bool FOLD = false>
__global__ __launch_bounds__(kThreads) void k_bicg_p_fused(int64_t N, int it, const T *__restrict__ r,
                                                           T *__restrict__ p, const T *__restrict__ v,
                                                           T *__restrict__ ph, T *__restrict__ rh,
                                                           const T *__restrict__ dinv,
                                                           const double *__restrict__ xr_partials, int xr_count,
                                                           KrylovScalars *sc) {
    using V = Vec16<T>;
    constexpr int W = V::W;
    const int64_t NV = N / W, stride = int64_t(gridDim.x) * kThreads;
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    typename V::type rv{}, po{}, vo{};
    auto load = [&] {
        rv = V::ld(r, i);
        po = V::ld(p, i);
        vo = V::ld(v, i);
    };
    if (i < NV) load();
    if (stopped(sc)) return;
    bool restart;
    double beta, omega;
    if (!bicg_p_scalars<T>(xr_partials, xr_count, sc, it, beta, omega, restart)) return;
    const T bt = T(beta), om = T(omega);
    while (i < NV) {
        const typename V::type pv = restart ? rv : rv + bt * (po - om * vo);
        V::st(p, i, pv);
        if (!FOLD) V::st(ph, i, V::ld(dinv, i) * pv);
        if (restart) V::st(rh, i, rv);
        i += stride;
        if (i < NV) load();
    }
    if (blockIdx.x == 0)
        for (int64_t i = NV * W + threadIdx.x; i < N; i += kThreads) {
            const T ri = r[i];
            const T pi = restart ? ri : ri + bt * (p[i] - om * v[i]);
            p[i] = pi;
            if (!FOLD) ph[i] = dinv[i] * pi;
            if (restart) rh[i] = ri;
        }
}

template <typename T, bool FOLD = false>
__global__ __launch_bounds__(kThreads) void k_bicg_s_fused(int64_t N, int it, const T *__restrict__ r,
                                                           const T *__restrict__ v, T *__restrict__ s,
                                                           T *__restrict__ sh, const T *__restrict__ dinv,
                                                           const double *__restrict__ sp_partials, int sp_count,
                                                           KrylovScalars *sc) {
    using V = Vec16<T>;
    constexpr int W = V::W;
    const int64_t NV = N / W, stride = int64_t(gridDim.x) * kThreads;
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    typename V::type rv{}, vv{};
    auto load = [&] {
        rv = V::ld(r, i);
        vv = V::ld(v, i);
    };
    if (i < NV) load();
    if (stopped(sc)) return;
    double alpha;
    if (!bicg_s_scalars(sp_partials, sp_count, sc, it, alpha)) return;
    const T al = T(alpha);
    while (i < NV) {
        const typename V::type sv = rv - al * vv;
        V::st(s, i, sv);
        if (!FOLD) V::st(sh, i, V::ld(dinv, i) * sv);
        i += stride;
        if (i < NV) load();
    }
    if (blockIdx.x == 0)
        for (int64_t i = NV * W + threadIdx.x; i < N; i += kThreads) {
            const T si = r[i] - al * v[i];
            s[i] = si;
            if (!FOLD) sh[i] = dinv[i] * si;
        }
}

template <typename T, bool FOLD = false>
__global__ __launch_bounds__(kThreads) void k_bicg_xr_fused(int64_t N, int it, T *__restrict__ x, T *__restrict__ r,
                                                            const T *__restrict__ rh, const T *__restrict__ ph,
                                                            const T *__restrict__ s, const T *__restrict__ sh,
                                                            const T *__restrict__ t,
                                                            const double *__restrict__ sp_partials, int sp_count,
                                                            double *xr_partials, KrylovScalars *sc) {
    using V = Vec16<T>;
    constexpr int W = V::W;
    const int64_t NV = N / W, stride = int64_t(gridDim.x) * kThreads;
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    typename V::type sv{}, xv{}, pv{}, tv{}, hv{};
    auto load = [&] {
        sv = V::ld(s, i);
        xv = V::ld(x, i);
        pv = V::ld(ph, i);
        tv = V::ld(t, i);
        hv = V::ld(rh, i);
    };
    if (i < NV) load();
    if (stopped(sc)) return;
    double tot[3];  // (t, s), (t, t), (s, s)
    sum_partials<3>(sp_partials, sp_count, tot);
    const double omega = bicg_omega<T>(tot);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->omega_pp[it & 1] = omega;
        sc->omega = omega;
    }
    const T al = T(sc->alpha_pp[it & 1]), om = T(omega);
    double d0 = 0.0, d1 = 0.0;
    while (i < NV) {
        V::st(x, i, xv + al * pv + om * (FOLD ? sv : V::ld(sh, i)));
        const typename V::type rv = sv - om * tv;
        V::st(r, i, rv);
#pragma unroll
        for (int c = 0; c < W; ++c) {
            d0 += double(hv[c]) * double(rv[c]);
            d1 += double(rv[c]) * double(rv[c]);
        }
        i += stride;
        if (i < NV) load();
    }
    if (blockIdx.x == 0)
        for (int64_t i = NV * W + threadIdx.x; i < N; i += kThreads) {
            const T si = s[i];
            x[i] += al * ph[i] + om * (FOLD ? si : sh[i]);
            const T ri = si - om * t[i];
            r[i] = ri;
            d0 += double(rh[i]) * double(ri);
            d1 += double(ri) * double(ri);
        }
    double vv[2] = {d0, d1};
    block_store_partials<2>(vv, xr_partials);
}

// Convergence, divergence and NaN flags after iteration it - 1 (one block; the next
// p-kernel repeats the same tests and also takes the restart decision).
__global__ __launch_bounds__(kThreads) void k_bicg_check(int it, const double *__restrict__ xr_partials,
                                                         int xr_count, KrylovScalars *sc, double rho_floor) {
    if (stopped(sc) || it == 0) return;
    double tot[2];
    sum_partials<2>(xr_partials, xr_count, tot);
    const BicgStart b = bicg_start_at(tot, sc, it, rho_floor);
    if (threadIdx.x == 0) bicg_publish_start(b, sc, it);
}

// CG's convergence and NaN flags after iteration it - 1 when the next SpMV would take
// them (one block; that SpMV repeats the test and publishes the other scalars).
__global__ __launch_bounds__(kThreads) void k_cg_check(int it, const double *__restrict__ rz_partials, int rz_count,
                                                       KrylovScalars *sc) {
    if (stopped(sc) || it == 0) return;
    double tot[2];
    sum_partials<2>(rz_partials, rz_count, tot);
    if (threadIdx.x != 0) return;
    sc->its = it;
    sc->rnorm2 = tot[1];
    if (!isfinite(tot[0]) || !isfinite(tot[1])) sc->breakdown = 2;
    else if (tot[1] <= sc->tol2) sc->converged = 1;
}

// ------------------------------------------------------------------ block Jacobi variants
// The same vector kernels with the node-block preconditioner: one thread per node,
// z_n = M_n r_n with M_n the inverse of node n's ND x ND diagonal block (row-major).
template <int ND, typename T>
__device__ __forceinline__ void node_block_apply(const T *__restrict__ M, int64_t n, const T r[ND], T z[ND]) {
    const T *m = M + int64_t(ND) * ND * n;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
        T a = T(0);
#pragma unroll
        for (int c = 0; c < ND; ++c) a += m[i * ND + c] * r[c];
        z[i] = a;
    }
}

template <int ND, typename T>
__global__ __launch_bounds__(kThreads) void k_kry_init_bj(int64_t Nn, int cg, const T *__restrict__ b,
                                                          T *__restrict__ x, T *__restrict__ r, T *__restrict__ rh,
                                                          T *__restrict__ p, T *__restrict__ v,
                                                          const T *__restrict__ M, double *partials) {
    double d0 = 0.0, d1 = 0.0;
    for (int64_t n = int64_t(blockIdx.x) * kThreads + threadIdx.x; n < Nn; n += int64_t(gridDim.x) * kThreads) {
        T bi[ND], zi[ND];
#pragma unroll
        for (int c = 0; c < ND; ++c) bi[c] = b[ND * n + c];
        if (cg) node_block_apply<ND>(M, n, bi, zi);
#pragma unroll
        for (int c = 0; c < ND; ++c) {
            const int64_t i = ND * n + c;
            x[i] = T(0);
            r[i] = bi[c];
            if (cg) {
                rh[i] = zi[c];
                p[i] = zi[c];
                d0 += double(bi[c]) * double(zi[c]);
            } else {
                rh[i] = bi[c];
                p[i] = T(0);
                v[i] = T(0);
                d0 += double(bi[c]) * double(bi[c]);
            }
            d1 += double(bi[c]) * double(bi[c]);
        }
    }
    double vv[2] = {d0, d1};
    block_store_partials<2>(vv, partials);
}

template <int ND, typename T>
__global__ __launch_bounds__(kThreads) void k_cg_xr_fused_bj(int64_t Nn, T *__restrict__ x, T *__restrict__ r,
                                                             T *__restrict__ z, const T *__restrict__ p,
                                                             const T *__restrict__ q, const T *__restrict__ M,
                                                             const double *__restrict__ pq_partials, int pq_count,
                                                             double *partials, KrylovScalars *sc, int it) {
    if (stopped(sc)) return;
    double pq[1];
    sum_partials<1>(pq_partials, pq_count, pq);
    if (!(pq[0] > 0.0) || !isfinite(pq[0])) {
        if (blockIdx.x == 0 && threadIdx.x == 0) sc->breakdown = 1;
        return;
    }
    const double alpha = sc->rho_pp[it & 1] / pq[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->alpha = alpha;
    const T al = T(alpha);
    double d0 = 0.0, d1 = 0.0;
    for (int64_t n = int64_t(blockIdx.x) * kThreads + threadIdx.x; n < Nn; n += int64_t(gridDim.x) * kThreads) {
        T ri[ND], zi[ND];
#pragma unroll
        for (int c = 0; c < ND; ++c) {
            const int64_t i = ND * n + c;
            x[i] += al * p[i];
            ri[c] = r[i] - al * q[i];
            r[i] = ri[c];
        }
        node_block_apply<ND>(M, n, ri, zi);
#pragma unroll
        for (int c = 0; c < ND; ++c) {
            z[ND * n + c] = zi[c];
            d0 += double(ri[c]) * double(zi[c]);
            d1 += double(ri[c]) * double(ri[c]);
        }
    }
    double v[2] = {d0, d1};
    block_store_partials<2>(v, partials);
}

template <int ND, typename T>
__global__ __launch_bounds__(kThreads) void k_bicg_p_bj(int64_t Nn, const T *__restrict__ r, T *__restrict__ p,
                                                        const T *__restrict__ v, T *__restrict__ ph,
                                                        T *__restrict__ rh, const T *__restrict__ M,
                                                        const KrylovScalars *sc) {
    if (stopped(sc)) return;
    const bool restart = sc->restart_at == sc->its;
    const double beta = (sc->its == 0 || restart) ? 0.0 : (sc->rho / sc->rho_old) * (sc->alpha / sc->omega);
    const T bt = T(beta), om = T(sc->omega);
    for (int64_t n = int64_t(blockIdx.x) * kThreads + threadIdx.x; n < Nn; n += int64_t(gridDim.x) * kThreads) {
        T pi[ND], zi[ND];
#pragma unroll
        for (int c = 0; c < ND; ++c) {
            const int64_t i = ND * n + c;
            const T ri = r[i];
            pi[c] = restart ? ri : ri + bt * (p[i] - om * v[i]);
            p[i] = pi[c];
            if (restart) rh[i] = ri;
        }
        node_block_apply<ND>(M, n, pi, zi);
#pragma unroll
        for (int c = 0; c < ND; ++c) ph[ND * n + c] = zi[c];
    }
}

template <int ND, typename T>
__global__ __launch_bounds__(kThreads) void k_bicg_s_bj(int64_t Nn, const T *__restrict__ r, const T *__restrict__ v,
                                                        T *__restrict__ s, T *__restrict__ sh,
                                                        const T *__restrict__ M, const KrylovScalars *sc) {
    if (stopped(sc)) return;
    const T al = T(sc->alpha);
    for (int64_t n = int64_t(blockIdx.x) * kThreads + threadIdx.x; n < Nn; n += int64_t(gridDim.x) * kThreads) {
        T si[ND], zi[ND];
#pragma unroll
        for (int c = 0; c < ND; ++c) {
            const int64_t i = ND * n + c;
            si[c] = r[i] - al * v[i];
            s[i] = si[c];
        }
        node_block_apply<ND>(M, n, si, zi);
#pragma unroll
        for (int c = 0; c < ND; ++c) sh[ND * n + c] = zi[c];
    }
}

// Krylov start with x0 = 0: r = rh = b, p = v = 0 (BiCGSTAB) or r = b, z = Dinv b,
// p = z (CG); reduces |b|^2 and the first rho.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_kry_init(int64_t N, int cg, const T *__restrict__ b,
                                                       T *__restrict__ x, T *__restrict__ r, T *__restrict__ rh,
                                                       T *__restrict__ p, T *__restrict__ v,
                                                       const T *__restrict__ dinv, double *partials,
                                                       KrylovScalars *sc, double rtol) {
    double d0 = 0.0, d1 = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x; i < N; i += int64_t(gridDim.x) * kThreads) {
        T bi = b[i];
        x[i] = T(0);
        r[i] = bi;
        if (cg) {
            T zi = dinv[i] * bi;
            rh[i] = zi;  // z
            p[i] = zi;
            d0 += double(bi) * double(zi);
        } else {
            rh[i] = bi;
            p[i] = T(0);
            v[i] = T(0);
            d0 += double(bi) * double(bi);
        }
        d1 += double(bi) * double(bi);
    }
    double vv[2] = {d0, d1};
    block_store_partials<2>(vv, partials);
}

__global__ __launch_bounds__(kThreads) void k_fin_init(int G, const double *__restrict__ partials,
                                                       KrylovScalars *sc, double rtol) {
    double tot[2];
    sum_partials<2>(partials, G, tot);
    if (threadIdx.x == 0) {
        sc->rho = tot[0];
        sc->rho_pp[0] = tot[0];
        sc->rho_pp[1] = tot[0];
        sc->rho_old = 1.0;
        sc->alpha = 1.0;
        sc->omega = 1.0;
        sc->beta = 0.0;
        sc->bnorm2 = tot[1];
        sc->rnorm2 = tot[1];
        sc->tol2 = rtol * rtol * tot[1];
        sc->its = 0;
        sc->rh2 = tot[1];
        sc->rmin2 = tot[1];
        sc->restart_at = -1;
        sc->alpha_pp[0] = sc->alpha_pp[1] = 1.0;
        sc->omega_pp[0] = sc->omega_pp[1] = 1.0;
        sc->rh2_pp[0] = sc->rh2_pp[1] = tot[1];
        sc->rmin2_pp[0] = sc->rmin2_pp[1] = tot[1];
        sc->breakdown = isfinite(tot[1]) ? 0 : 2;
        sc->converged = (tot[1] == 0.0) ? 1 : 0;
    }
}

// ------------------------------------------------------------------ vector helpers
__global__ __launch_bounds__(kThreads) void k_dot_self(int64_t N, const double *__restrict__ r, double *partials) {
    double d = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x; i < N; i += int64_t(gridDim.x) * kThreads)
        d += r[i] * r[i];
    double v[1] = {d};
    block_store_partials<1>(v, partials);
}

__global__ __launch_bounds__(kThreads) void k_fin_dot(int G, const double *__restrict__ partials, double *out) {
    double tot[1];
    sum_partials<1>(partials, G, tot);
    if (threadIdx.x == 0) *out = tot[0];
}

template <typename TO, typename TI>
__global__ __launch_bounds__(kThreads) void k_scale_cast(int64_t n, const TI *__restrict__ in, TO *__restrict__ out,
                                                         double alpha) {
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) out[i] = TO(alpha * double(in[i]));
}

template <typename TI>
__global__ __launch_bounds__(kThreads) void k_axpy_f64(int64_t n, const TI *__restrict__ x, double *__restrict__ y) {
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) y[i] += double(x[i]);
}

__global__ __launch_bounds__(kThreads) void k_set_dirichlet(int64_t n, const uint8_t *__restrict__ mask,
                                                            double *__restrict__ u, const double *__restrict__ u0,
                                                            const double *__restrict__ g, double lam) {
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n && mask[i]) u[i] = u0[i] + lam * (g[i] - u0[i]);
}

__global__ __launch_bounds__(kThreads) void k_dirichlet_increment(int64_t n, const uint8_t *__restrict__ mask,
                                                                  const double *__restrict__ u,
                                                                  const double *__restrict__ u0,
                                                                  const double *__restrict__ g, double lam,
                                                                  double *__restrict__ delta) {
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) delta[i] = mask[i] ? (u0[i] + lam * (g[i] - u0[i]) - u[i]) : 0.0;
}

__global__ __launch_bounds__(kThreads) void k_neg_sum(int64_t n, const double *__restrict__ a,
                                                      const double *__restrict__ b, double *__restrict__ out) {
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) out[i] = -(a[i] + b[i]);
}

__global__ __launch_bounds__(kThreads) void k_mask_copy(int64_t n, const uint8_t *__restrict__ mask,
                                                        const double *__restrict__ in, double *__restrict__ out) {
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) out[i] = (mask && mask[i]) ? 0.0 : in[i];
}

__global__ __launch_bounds__(kThreads) void k_sub(int64_t n, const double *__restrict__ a,
                                                  const double *__restrict__ b, double *__restrict__ out) {
    int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) out[i] = a[i] - b[i];
}

// ------------------------------------------------------------------ pattern export
template <int ND>
__global__ __launch_bounds__(kThreads) void k_export_cols(int64_t nnzb, const int64_t *__restrict__ node_ptr,
                                                          const int32_t *__restrict__ node_nb,
                                                          const int32_t *__restrict__ blk_row,
                                                          const int32_t *__restrict__ mirror,
                                                          const int64_t *__restrict__ row_ptr,
                                                          int32_t *__restrict__ col_idx, int32_t *__restrict__ tperm) {
    int64_t t = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (t >= nnzb * ND * ND) return;
    int64_t kb = t / (ND * ND);
    int r = int(t - kb * ND * ND);
    int i = r / ND, k = r % ND;
    int64_t n = blk_row[kb], m = node_nb[kb];
    int64_t pos = row_ptr[ND * n + i] + ND * (kb - node_ptr[n]) + k;
    if (col_idx) col_idx[pos] = int32_t(ND * m + k);
    if (tperm) tperm[pos] = int32_t(row_ptr[ND * m + k] + ND * (mirror[kb] - node_ptr[m]) + i);
}

template <int ND>
__global__ __launch_bounds__(kThreads) void k_export_slots(int64_t Ne, const int32_t *__restrict__ conn,
                                                           const int32_t *__restrict__ bslot,
                                                           const int64_t *__restrict__ node_ptr,
                                                           const int64_t *__restrict__ row_ptr,
                                                           int32_t *__restrict__ slot) {
    constexpr int Nd = 8 * ND;
    int64_t t = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (t >= Ne * Nd * Nd) return;
    int64_t e = t / (Nd * Nd);
    int r = int(t - e * Nd * Nd);
    int p = r / Nd, q = r % Nd;
    int a = p / ND, i = p % ND, b = q / ND, k = q % ND;
    int64_t n = conn[8 * e + a];
    int64_t kb = bslot[e * 64 + a * 8 + b];
    slot[t] = int32_t(row_ptr[ND * n + i] + ND * (kb - node_ptr[n]) + k);
}

template <int ND>
__global__ __launch_bounds__(kThreads) void k_export_diag(int64_t N, const int32_t *__restrict__ bdiag,
                                                          const int64_t *__restrict__ node_ptr,
                                                          const int64_t *__restrict__ row_ptr,
                                                          int64_t *__restrict__ diag) {
    int64_t d = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (d >= N) return;
    int64_t n = d / ND;
    int i = int(d - n * ND);
    diag[d] = row_ptr[d] + ND * (bdiag[n] - node_ptr[n]) + i;
}

}  // namespace

int krylov_grid(const fem_handle *h) {
    // Largest persistent grid: 8 resident blocks of 4 waves per CU (8 waves per SIMD).
    return 8 * h->num_cus;
}

// Grid of the Krylov vector kernels.  Their blocks store one partial each, and every
// block of the next kernel sums all of them, so at most 4 blocks per CU, and no more than
// give each thread one 16-byte access: 180 blocks at 92k dofs, 1,024 at 3.1M.  Against
// 1,024 everywhere, with the register-move reductions: 2.2 us less per CG iteration at
// 212k dofs (33.1 instead of 35.4 us), 3.4 us per BiCGSTAB iteration at 207k.
static int krylov_vec_grid(const fem_handle *h) {
    return int(std::max<int64_t>(1, std::min<int64_t>(4 * h->num_cus, (h->g.N + 2 * kThreads - 1) / (2 * kThreads))));
}

// Persistent grid of a kernel: the blocks that can be resident at once (runtime
// occupancy of this kernel variant), a multiple of the 8 XCDs.
template <typename K>
static int resident_grid(const fem_handle *h, K kernel) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    int G = std::min(per_cu, 8) * h->num_cus;
    return std::max(8, (G / 8) * 8);
}

// Grid of k_spmv_nodes, by the size of the stored values: two blocks per CU for 8-byte
// values (100^3: 352 us; three or four 385 us, one node more in flight 374 us), three
// for 4-byte values (100^3: 183.6 us; two 217.5 us, seven 207.7 us).  Products with one
// dof per node are too short to be bound by bytes (50x50x10: 4.8 us with eight, 6.3 us
// with two).
template <int ND, typename TV>
static int spmv_grid(const fem_handle *h) {
    return (ND == 1 ? 8 : (sizeof(TV) == 8 ? 2 : 3)) * h->num_cus;
}

template <int ND, typename T>
static void spmv_launch(const fem_handle *h, const T *values, int transpose, const T *x, T *y, T alpha, T beta,
                        hipStream_t s) {
    const Graph &g = h->g;
    if (transpose)
        hipLaunchKernelGGL((k_spmv_t<ND, T>), dim3((grid_for(g.Nn, kThreads / 32) + 7) / 8 * 8), dim3(kThreads), 0, s,
                           g.Nn, g.node_ptr, g.node_nb, g.mirror, values, x, y, alpha, beta);
    else if (g.node_dnb)
        hipLaunchKernelGGL((k_spmv_nodes<ND, 0, T, true>), dim3(spmv_grid<ND, T>(h)), dim3(kThreads), 0, s, g.Nn,
                           g.node_ptr, g.node_nb, g.node_dnb, values, x, y, nullptr, alpha, beta, nullptr, nullptr, 0,
                           int(g.max_deg > kSpmvGroup), GatherIn<T>());
    else
        hipLaunchKernelGGL((k_spmv_nodes<ND, 0, T, false>), dim3(spmv_grid<ND, T>(h)), dim3(kThreads), 0, s, g.Nn,
                           g.node_ptr, g.node_nb, g.node_dnb, values, x, y, nullptr, alpha, beta, nullptr, nullptr, 0,
                           int(g.max_deg > kSpmvGroup), GatherIn<T>());
}

template <typename T>
void launch_spmv(const fem_handle *h, const T *values, int transpose, const T *x, T *y, T alpha, T beta,
                 hipStream_t s) {
    const Graph &g = h->g;
    if (g.Nn == 0) return;
    if (g.nd == 1) spmv_launch<1, T>(h, values, transpose, x, y, alpha, beta, s);
    else spmv_launch<3, T>(h, values, transpose, x, y, alpha, beta, s);
    FEM_HIP(hipGetLastError());
}

template <typename T>
void launch_spmv_sym(const fem_handle *h, const T *values, const T *x, T *y, T alpha, T beta, hipStream_t s) {
    const Graph &g = h->g;
    if (g.Nn == 0) return;
#define FEM_SYM0(ND)                                                                                            \
    hipLaunchKernelGGL((k_spmv_sym<ND, 4, 0, T>), dim3(resident_grid(h, k_spmv_sym<ND, 4, 0, T>)), dim3(kThreads),  \
                       0, s, g.Nn, g.node_ptr, g.up_base, g.node_nb, g.lo_val, values, x, y, nullptr, alpha, beta,  \
                       nullptr, nullptr, 0)
    if (g.nd == 1) FEM_SYM0(1);
    else FEM_SYM0(3);
#undef FEM_SYM0
    FEM_HIP(hipGetLastError());
}
template void launch_spmv_sym<float>(const fem_handle *, const float *, const float *, float *, float, float,
                                     hipStream_t);
template void launch_spmv_sym<double>(const fem_handle *, const double *, const double *, double *, double, double,
                                      hipStream_t);

template <typename T>
void kry_bicg_init(const fem_handle *h, const KrylovVecs<T> &k, const T *b, double rtol, hipStream_t s) {
    if (k.bj) {
        if (h->g.nd == 1)
            hipLaunchKernelGGL((k_kry_init_bj<1, T>), dim3(krylov_vec_grid(h)), dim3(kThreads), 0, s, h->g.Nn, 0, b, k.x,
                               k.r, k.rh, k.p, k.v, k.dinv, k.partials);
        else
            hipLaunchKernelGGL((k_kry_init_bj<3, T>), dim3(krylov_vec_grid(h)), dim3(kThreads), 0, s, h->g.Nn, 0, b, k.x,
                               k.r, k.rh, k.p, k.v, k.dinv, k.partials);
    } else {
        hipLaunchKernelGGL((k_kry_init<T>), dim3(krylov_vec_grid(h)), dim3(kThreads), 0, s, h->g.N, 0, b, k.x, k.r, k.rh,
                           k.p, k.v, k.dinv, k.partials, k.sc, rtol);
    }
    hipLaunchKernelGGL(k_fin_init, dim3(1), dim3(kThreads), 0, s, krylov_vec_grid(h), k.partials, k.sc, rtol);
    FEM_HIP(hipGetLastError());
}

template <typename T>
void kry_cg_init(const fem_handle *h, const KrylovVecs<T> &k, const T *b, double rtol, hipStream_t s) {
    // CG keeps z in the slot of rh
    if (k.bj) {
        if (h->g.nd == 1)
            hipLaunchKernelGGL((k_kry_init_bj<1, T>), dim3(krylov_vec_grid(h)), dim3(kThreads), 0, s, h->g.Nn, 1, b, k.x,
                               k.r, k.rh, k.p, k.v, k.dinv, k.partials);
        else
            hipLaunchKernelGGL((k_kry_init_bj<3, T>), dim3(krylov_vec_grid(h)), dim3(kThreads), 0, s, h->g.Nn, 1, b, k.x,
                               k.r, k.rh, k.p, k.v, k.dinv, k.partials);
    } else {
        hipLaunchKernelGGL((k_kry_init<T>), dim3(krylov_vec_grid(h)), dim3(kThreads), 0, s, h->g.N, 1, b, k.x, k.r, k.rh,
                           k.p, k.v, k.dinv, k.partials, k.sc, rtol);
    }
    hipLaunchKernelGGL(k_fin_init, dim3(1), dim3(kThreads), 0, s, krylov_vec_grid(h), k.partials, k.sc, rtol);
    FEM_HIP(hipGetLastError());
}

// Launches the fused SpMV (partials into k.partials) and, unless the caller folds it
// into its next kernel, the one-block finalize; returns the SpMV grid size.
template <int ND, int MODE, typename T, typename TV = T, int GATHER = GATHER_X>
static int kry_spmv_launch(const fem_handle *h, const T *x, T *y, const T *w0, const KrylovVecs<T> &k, int cg,
                           const TV *values, bool finalize, hipStream_t s, double *partials, GatherIn<T> gi) {
    const Graph &g = h->g;
    int G;
    if (k.layout == LAYOUT_SYM) {
        if constexpr (std::is_same<T, TV>::value && GATHER == GATHER_X) {
            G = resident_grid(h, k_spmv_sym<ND, 4, MODE, T>);
            hipLaunchKernelGGL((k_spmv_sym<ND, 4, MODE, T>), dim3(G), dim3(kThreads), 0, s, g.Nn, g.node_ptr,
                               g.up_base, g.node_nb, g.lo_val, values, x, y, w0, T(1), T(0), partials, k.sc, cg);
        } else {
            throw Error(FEM_EINVAL, "the symmetric block layout takes values of the vector type");
        }
    } else if (g.node_dnb) {
        G = spmv_grid<ND, TV>(h);
        hipLaunchKernelGGL((k_spmv_nodes<ND, MODE, T, true, TV, GATHER>), dim3(G), dim3(kThreads), 0, s, g.Nn,
                           g.node_ptr, g.node_nb, g.node_dnb, values, x, y, w0, T(1), T(0), partials, k.sc, cg,
                           int(g.max_deg > kSpmvGroup), gi);
    } else {
        G = spmv_grid<ND, TV>(h);
        hipLaunchKernelGGL((k_spmv_nodes<ND, MODE, T, false, TV, GATHER>), dim3(G), dim3(kThreads), 0, s, g.Nn,
                           g.node_ptr, g.node_nb, g.node_dnb, values, x, y, w0, T(1), T(0), partials, k.sc, cg,
                           int(g.max_deg > kSpmvGroup), gi);
    }
    if (finalize) {
        if (MODE == 1) hipLaunchKernelGGL(k_fin_alpha, dim3(1), dim3(kThreads), 0, s, G, partials, k.sc, cg);
        else hipLaunchKernelGGL(k_fin_omega, dim3(1), dim3(kThreads), 0, s, G, partials, k.sc);
    }
    return G;
}

// The Krylov SpMV on the solve's operator: k.A, or the FP32 tangent k.A32 under FP64
// vectors (products and sums in FP64).
template <typename T, int MODE, int GATHER = GATHER_X>
static int kry_spmv(const fem_handle *h, const T *x, T *y, const T *w0, const KrylovVecs<T> &k, int cg,
                    const T *values, hipStream_t s, bool finalize = true, double *partials = nullptr,
                    GatherIn<T> gi = GatherIn<T>()) {
    if (!partials) partials = k.partials;
    if constexpr (sizeof(T) == 8) {
        if (k.A32) {
            if (h->g.nd == 1)
                return kry_spmv_launch<1, MODE, T, float, GATHER>(h, x, y, w0, k, cg, k.A32, finalize, s, partials, gi);
            return kry_spmv_launch<3, MODE, T, float, GATHER>(h, x, y, w0, k, cg, k.A32, finalize, s, partials, gi);
        }
    }
    if (h->g.nd == 1)
        return kry_spmv_launch<1, MODE, T, T, GATHER>(h, x, y, w0, k, cg, values, finalize, s, partials, gi);
    return kry_spmv_launch<3, MODE, T, T, GATHER>(h, x, y, w0, k, cg, values, finalize, s, partials, gi);
}

// Whether an iteration forms p (and BiCGSTAB's s) inside the SpMV's gathers instead of in
// vector kernels of their own.  Each formed vector saves a launch (3 to 6 us while the
// vectors are small) and costs one or two more gathers per block, which grow with the
// mesh.  Time per iteration, vector kernels -> gathers (3 dofs per node, FP64):
//   CG (one more gather)         N = 27,783: 15.0 -> 12.0 us; 206,763: 32.7 -> 30.7; 680,943: 106 -> 114
//   CG, FP32                     206,763: 22.8 -> 20.7; 680,943: 50.4 -> 49.3; 1,594,323: 130 -> 134
//   BiCGSTAB (two and one more)  N = 27,783: 27.1 -> 20.9 us; 89,373: 37.8 -> 36.8; 206,763: 60.7 -> 63.7
//   BiCGSTAB, FP32               27,783: 25.6 -> 20.7; 89,373: 31.5 -> 33.4
// With one dof per node: CG N = 29,791: 16.2 -> 14.6, 226,981: 27.2 -> 29.0; BiCGSTAB
// 29,791: 30.6 -> 27.1, 226,981: 53.8 -> 61.0.
template <typename T>
static bool krylov_gathers(const fem_handle *h, const KrylovVecs<T> &k, bool cg) {
    const int64_t limit = cg ? (h->g.nd == 1 ? 100000 : 300000) : 60000;
    return k.layout == LAYOUT_CSR && h->g.N <= limit;
}

template <typename T>
int kry_spmv_q(const fem_handle *h, const KrylovVecs<T> &k, hipStream_t s) {
    return kry_spmv<T, 1>(h, k.p, k.v, k.p, k, 1, k.A, s, false);
}

int krylov_vec_grid_of(const fem_handle *h) { return krylov_vec_grid(h); }

// p = z + beta p from the (r, z) and |r|^2 partials in k.partials2 (krylov_vec_grid of them).
template <typename T>
void kry_cg_p_update(const fem_handle *h, const KrylovVecs<T> &k, int it, hipStream_t s) {
    const int G = krylov_vec_grid(h);
    hipLaunchKernelGGL((k_cg_p_fused<T>), dim3(G), dim3(kThreads), 0, s, h->g.N, k.rh, k.p, k.partials2, G, k.sc, it);
    FEM_HIP(hipGetLastError());
}

// y = alpha K x + beta y inside a Krylov loop: skipped once sc reports convergence.
template <typename T>
void launch_spmv_sc(const fem_handle *h, const T *values, const T *x, T *y, T alpha, T beta, const KrylovScalars *sc,
                    hipStream_t s) {
    const Graph &g = h->g;
    if (g.N == 0) return;
    KrylovScalars *scw = const_cast<KrylovScalars *>(sc);
#define FEM_SPMV_SC(ND, D16)                                                                                       \
    hipLaunchKernelGGL((k_spmv_nodes<ND, 0, T, D16>),                                         \
                       dim3(spmv_grid<ND, T>(h)), dim3(kThreads), 0, \
                       s, g.Nn, g.node_ptr, g.node_nb, g.node_dnb, values, x, y, nullptr, alpha, beta, nullptr,   \
                       scw, 0, int(g.max_deg > kSpmvGroup))
    if (g.nd == 1) {
        if (g.node_dnb) FEM_SPMV_SC(1, true);
        else FEM_SPMV_SC(1, false);
    } else {
        if (g.node_dnb) FEM_SPMV_SC(3, true);
        else FEM_SPMV_SC(3, false);
    }
#undef FEM_SPMV_SC
    FEM_HIP(hipGetLastError());
}

template <typename T>
void kry_bicg_iter(const fem_handle *h, const KrylovVecs<T> &k, int it, hipStream_t s, hipEvent_t *ev) {
    const int64_t N = h->g.N;
    const T *A = k.A;
    const int64_t Nn = h->g.Nn;
    if (!k.bj) {
        dim3 grid(krylov_vec_grid(h)), blk(kThreads);
        // folded Jacobi: the operator is K D^{-1} and the SpMVs take p and s directly
        if (k.fold && krylov_gathers(h, k, false)) {
            // three kernels; p and v alternate between two buffers each (ph and sh are free),
            // since blocks still gather the old ones while others write the new
            T *pb[2] = {k.p, k.ph}, *vb[2] = {k.v, k.sh};
            const int o = it & 1, n = 1 - o;
            double *sp = k.partials + krylov_grid(h);  // of the second SpMV, which reads the first one's
            GatherIn<T> gi;
            gi.b = pb[o];
            gi.c = vb[o];
            gi.out = pb[n];
            gi.rh = k.rh;
            gi.partials = k.partials2;
            gi.count = int(grid.x);
            gi.it = it;
            if (ev) FEM_HIP(hipEventRecord(ev[0], s));
            const int G1 = kry_spmv<T, 1, GATHER_BICG_P>(h, k.r, vb[n], nullptr, k, 0, A, s, false, k.partials, gi);
            if (ev) FEM_HIP(hipEventRecord(ev[1], s));
            GatherIn<T> gs;
            gs.b = vb[n];
            gs.out = k.s;
            gs.partials = k.partials;
            gs.count = G1;
            gs.it = it;
            if (ev) FEM_HIP(hipEventRecord(ev[2], s));
            const int G2 = kry_spmv<T, 2, GATHER_BICG_S>(h, k.r, k.t, nullptr, k, 0, A, s, false, sp, gs);
            if (ev) FEM_HIP(hipEventRecord(ev[3], s));
            hipLaunchKernelGGL((k_bicg_xr_fused<T, true>), grid, blk, 0, s, N, it, k.x, k.r, k.rh, pb[n], k.s, k.s, k.t,
                               sp, G2, k.partials2, k.sc);
            FEM_HIP(hipGetLastError());
            return;
        }
        T *ph = k.fold ? k.p : k.ph, *sh = k.fold ? k.s : k.sh;
        if (k.fold)
            hipLaunchKernelGGL((k_bicg_p_fused<T, true>), grid, blk, 0, s, N, it, k.r, k.p, k.v, ph, k.rh, k.dinv,
                               k.partials2, int(grid.x), k.sc);
        else
            hipLaunchKernelGGL((k_bicg_p_fused<T, false>), grid, blk, 0, s, N, it, k.r, k.p, k.v, ph, k.rh, k.dinv,
                               k.partials2, int(grid.x), k.sc);
        if (ev) FEM_HIP(hipEventRecord(ev[0], s));
        int G = kry_spmv<T, 1>(h, ph, k.v, k.rh, k, 0, A, s, false);
        if (ev) FEM_HIP(hipEventRecord(ev[1], s));
        if (k.fold)
            hipLaunchKernelGGL((k_bicg_s_fused<T, true>), grid, blk, 0, s, N, it, k.r, k.v, k.s, sh, k.dinv,
                               k.partials, G, k.sc);
        else
            hipLaunchKernelGGL((k_bicg_s_fused<T, false>), grid, blk, 0, s, N, it, k.r, k.v, k.s, sh, k.dinv,
                               k.partials, G, k.sc);
        if (ev) FEM_HIP(hipEventRecord(ev[2], s));
        G = kry_spmv<T, 2>(h, sh, k.t, k.s, k, 0, A, s, false);
        if (ev) FEM_HIP(hipEventRecord(ev[3], s));
        if (k.fold)
            hipLaunchKernelGGL((k_bicg_xr_fused<T, true>), grid, blk, 0, s, N, it, k.x, k.r, k.rh, ph, k.s, sh, k.t,
                               k.partials, G, k.partials2, k.sc);
        else
            hipLaunchKernelGGL((k_bicg_xr_fused<T, false>), grid, blk, 0, s, N, it, k.x, k.r, k.rh, ph, k.s, sh, k.t,
                               k.partials, G, k.partials2, k.sc);
        FEM_HIP(hipGetLastError());
        return;
    }
    // block Jacobi: separate vector kernels with one-block finalizes
    dim3 grid(krylov_grid(h)), blk(kThreads);
    if (h->g.nd == 1) hipLaunchKernelGGL((k_bicg_p_bj<1, T>), grid, blk, 0, s, Nn, k.r, k.p, k.v, k.ph, k.rh, k.dinv, k.sc);
    else hipLaunchKernelGGL((k_bicg_p_bj<3, T>), grid, blk, 0, s, Nn, k.r, k.p, k.v, k.ph, k.rh, k.dinv, k.sc);
    if (ev) FEM_HIP(hipEventRecord(ev[0], s));
    kry_spmv<T, 1>(h, k.ph, k.v, k.rh, k, 0, A, s);
    if (ev) FEM_HIP(hipEventRecord(ev[1], s));
    if (h->g.nd == 1) hipLaunchKernelGGL((k_bicg_s_bj<1, T>), grid, blk, 0, s, Nn, k.r, k.v, k.s, k.sh, k.dinv, k.sc);
    else hipLaunchKernelGGL((k_bicg_s_bj<3, T>), grid, blk, 0, s, Nn, k.r, k.v, k.s, k.sh, k.dinv, k.sc);
    if (ev) FEM_HIP(hipEventRecord(ev[2], s));
    kry_spmv<T, 2>(h, k.sh, k.t, k.s, k, 0, A, s);
    if (ev) FEM_HIP(hipEventRecord(ev[3], s));
    hipLaunchKernelGGL((k_bicg_xr<T>), grid, blk, 0, s, N, k.x, k.r, k.rh, k.ph, k.s, k.sh, k.t, k.partials, k.sc);
    hipLaunchKernelGGL(k_fin_bicg_xr, dim3(1), blk, 0, s, int(grid.x), k.partials, k.sc);
    FEM_HIP(hipGetLastError());
}

template <typename T>
void kry_bicg_check(const fem_handle *h, const KrylovVecs<T> &k, int it, hipStream_t s) {
    if (k.bj) return;  // the unfused iteration finalizes its own scalars
    hipLaunchKernelGGL(k_bicg_check, dim3(1), dim3(kThreads), 0, s, it, k.partials2, krylov_vec_grid(h), k.sc,
                       sizeof(T) == 4 ? kRhoFloorF32 : 1e-9);
    FEM_HIP(hipGetLastError());
}

// One CG iteration in three kernels: q = K p with (p, q) partials; the x/r/z update
// with alpha taken from those partials; the p update with beta taken from the
// (r, z) partials.  The two partial buffers alternate so that no kernel overwrites
// partials that blocks of the same kernel are still reading.
template <typename T>
void kry_cg_iter(const fem_handle *h, const KrylovVecs<T> &k, int it, hipStream_t s, hipEvent_t *ev) {
    const int64_t N = h->g.N;
    dim3 grid(krylov_vec_grid(h)), blk(kThreads);
    const T *A = k.A;
    // slots: z = rh, q = v; p alternates between two buffers when the SpMV forms it
    const bool gathers = krylov_gathers(h, k, true);
    T *p = k.p;
    int G;
    if (ev) FEM_HIP(hipEventRecord(ev[0], s));
    if (gathers) {
        T *pb[2] = {k.p, k.ph};
        p = pb[1 - (it & 1)];
        GatherIn<T> gi;
        gi.b = pb[it & 1];
        gi.out = p;
        gi.partials = k.partials2;
        gi.count = int(grid.x);
        gi.it = it;
        G = kry_spmv<T, 1, GATHER_CG_P>(h, k.rh, k.v, nullptr, k, 1, A, s, false, k.partials, gi);
    } else {
        G = kry_spmv<T, 1>(h, k.p, k.v, k.p, k, 1, A, s, false);
    }
    if (ev) FEM_HIP(hipEventRecord(ev[1], s));
    if (!k.bj)
        hipLaunchKernelGGL((k_cg_xr_fused<T>), grid, blk, 0, s, N, k.x, k.r, k.rh, p, k.v, k.dinv, k.partials, G,
                           k.partials2, k.sc, it);
    else if (h->g.nd == 1)
        hipLaunchKernelGGL((k_cg_xr_fused_bj<1, T>), grid, blk, 0, s, h->g.Nn, k.x, k.r, k.rh, p, k.v, k.dinv,
                           k.partials, G, k.partials2, k.sc, it);
    else
        hipLaunchKernelGGL((k_cg_xr_fused_bj<3, T>), grid, blk, 0, s, h->g.Nn, k.x, k.r, k.rh, p, k.v, k.dinv,
                           k.partials, G, k.partials2, k.sc, it);
    if (!gathers)
        hipLaunchKernelGGL((k_cg_p_fused<T>), grid, blk, 0, s, N, k.rh, k.p, k.partials2, int(grid.x), k.sc, it);
    FEM_HIP(hipGetLastError());
}

template <typename T>
void kry_cg_check(const fem_handle *h, const KrylovVecs<T> &k, int it, hipStream_t s) {
    if (!krylov_gathers(h, k, true)) return;  // the p kernel has tested already
    hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(kThreads), 0, s, it, k.partials2, krylov_vec_grid(h), k.sc);
    FEM_HIP(hipGetLastError());
}

template void kry_bicg_init<float>(const fem_handle *, const KrylovVecs<float> &, const float *, double, hipStream_t);
template void kry_bicg_init<double>(const fem_handle *, const KrylovVecs<double> &, const double *, double,
                                    hipStream_t);
template void kry_cg_init<float>(const fem_handle *, const KrylovVecs<float> &, const float *, double, hipStream_t);
template void kry_cg_init<double>(const fem_handle *, const KrylovVecs<double> &, const double *, double, hipStream_t);
template void kry_bicg_iter<float>(const fem_handle *, const KrylovVecs<float> &, int, hipStream_t, hipEvent_t *);
template void kry_bicg_iter<double>(const fem_handle *, const KrylovVecs<double> &, int, hipStream_t, hipEvent_t *);
template void kry_bicg_check<float>(const fem_handle *, const KrylovVecs<float> &, int, hipStream_t);
template void kry_bicg_check<double>(const fem_handle *, const KrylovVecs<double> &, int, hipStream_t);
template void kry_cg_check<float>(const fem_handle *, const KrylovVecs<float> &, int, hipStream_t);
template void kry_cg_check<double>(const fem_handle *, const KrylovVecs<double> &, int, hipStream_t);
template int kry_spmv_q<float>(const fem_handle *, const KrylovVecs<float> &, hipStream_t);
template int kry_spmv_q<double>(const fem_handle *, const KrylovVecs<double> &, hipStream_t);
template void kry_cg_p_update<float>(const fem_handle *, const KrylovVecs<float> &, int, hipStream_t);
template void kry_cg_p_update<double>(const fem_handle *, const KrylovVecs<double> &, int, hipStream_t);
template void launch_spmv_sc<float>(const fem_handle *, const float *, const float *, float *, float, float,
                                    const KrylovScalars *, hipStream_t);
template void launch_spmv_sc<double>(const fem_handle *, const double *, const double *, double *, double, double,
                                     const KrylovScalars *, hipStream_t);
template void kry_cg_iter<float>(const fem_handle *, const KrylovVecs<float> &, int, hipStream_t, hipEvent_t *);
template void kry_cg_iter<double>(const fem_handle *, const KrylovVecs<double> &, int, hipStream_t, hipEvent_t *);
template void launch_spmv<float>(const fem_handle *, const float *, int, const float *, float *, float, float,
                                 hipStream_t);
template void launch_spmv<double>(const fem_handle *, const double *, int, const double *, double *, double, double,
                                  hipStream_t);

void launch_norm2_free(const fem_handle *h, const double *r, double *partials, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_dot_self, dim3(krylov_vec_grid(h)), dim3(kThreads), 0, s, h->g.N, r, partials);
    hipLaunchKernelGGL(k_fin_dot, dim3(1), dim3(kThreads), 0, s, krylov_vec_grid(h), partials, out);
    FEM_HIP(hipGetLastError());
}

template <typename TO, typename TI>
void launch_scale_cast(const TI *in, TO *out, double alpha, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL((k_scale_cast<TO, TI>), dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, in, out, alpha);
    FEM_HIP(hipGetLastError());
}
template void launch_scale_cast<float, double>(const double *, float *, double, int64_t, hipStream_t);
template void launch_scale_cast<double, double>(const double *, double *, double, int64_t, hipStream_t);
template void launch_scale_cast<double, float>(const float *, double *, double, int64_t, hipStream_t);

// Right point-Jacobi scaling folded into the stored tangent: every value of column
// dof j is multiplied by dinv[j], so BiCGSTAB runs on K D^{-1} (the same iterates as
// right preconditioning with D, without the D^{-1} p and D^{-1} s vectors), and its
// iterate y maps back as x = D^{-1} y.  One 32-lane group per node, lane = block.
template <int ND, typename T>
__global__ __launch_bounds__(kThreads) void k_scale_columns(int64_t Nn, const int64_t *__restrict__ node_ptr,
                                                            const int32_t *__restrict__ node_nb,
                                                            T *__restrict__ values, const T *__restrict__ dinv) {
    constexpr int G = 32;
    const int lane = threadIdx.x % G;
    for (int64_t n = (int64_t(blockIdx.x) * kThreads + threadIdx.x) / G; n < Nn;
         n += int64_t(gridDim.x) * (kThreads / G)) {
        const int64_t b0 = node_ptr[n];
        const int deg = int(node_ptr[n + 1] - b0);
        for (int l = lane; l < deg; l += G) {
            const int64_t m = node_nb[b0 + l];
            T d[ND];
#pragma unroll
            for (int c = 0; c < ND; ++c) d[c] = dinv[ND * m + c];
            T *vb = values + int64_t(ND) * ND * b0 + ND * l;
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int c = 0; c < ND; ++c) vb[int64_t(i) * ND * deg + c] *= d[c];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_mul_inplace(int64_t n, T *__restrict__ x, const T *__restrict__ d) {
    for (int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x; i < n; i += int64_t(gridDim.x) * kThreads)
        x[i] *= d[i];
}

template <typename T>
void launch_scale_columns(const fem_handle *h, T *values, const T *dinv, hipStream_t s) {
    const Graph &g = h->g;
    if (g.Nn == 0) return;
    dim3 grid(grid_for(g.Nn, kThreads / 32));
    if (g.nd == 1)
        hipLaunchKernelGGL((k_scale_columns<1, T>), grid, dim3(kThreads), 0, s, g.Nn, g.node_ptr, g.node_nb, values,
                           dinv);
    else
        hipLaunchKernelGGL((k_scale_columns<3, T>), grid, dim3(kThreads), 0, s, g.Nn, g.node_ptr, g.node_nb, values,
                           dinv);
    FEM_HIP(hipGetLastError());
}
template void launch_scale_columns<float>(const fem_handle *, float *, const float *, hipStream_t);
template void launch_scale_columns<double>(const fem_handle *, double *, const double *, hipStream_t);

template <typename T>
void launch_mul_inplace(T *x, const T *d, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL((k_mul_inplace<T>), dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, x, d);
    FEM_HIP(hipGetLastError());
}
template void launch_mul_inplace<float>(float *, const float *, int64_t, hipStream_t);
template void launch_mul_inplace<double>(double *, const double *, int64_t, hipStream_t);

template <typename TI>
void launch_axpy_to_f64(const TI *x, double *y, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL((k_axpy_f64<TI>), dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, x, y);
    FEM_HIP(hipGetLastError());
}
template void launch_axpy_to_f64<float>(const float *, double *, int64_t, hipStream_t);
template void launch_axpy_to_f64<double>(const double *, double *, int64_t, hipStream_t);

void launch_set_dirichlet(const fem_handle *h, double *u, const double *u0, const double *g, double lam,
                          hipStream_t s) {
    if (h->g.N == 0) return;
    hipLaunchKernelGGL(k_set_dirichlet, dim3(grid_for(h->g.N, kThreads)), dim3(kThreads), 0, s, h->g.N, h->m.mask, u,
                       u0, g, lam);
    FEM_HIP(hipGetLastError());
}

void launch_dirichlet_increment(const fem_handle *h, const double *u, const double *u0, const double *g, double lam,
                                double *delta, hipStream_t s) {
    if (h->g.N == 0) return;
    hipLaunchKernelGGL(k_dirichlet_increment, dim3(grid_for(h->g.N, kThreads)), dim3(kThreads), 0, s, h->g.N,
                       h->m.mask, u, u0, g, lam, delta);
    FEM_HIP(hipGetLastError());
}

void launch_neg_sum(const double *a, const double *b, double *out, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_neg_sum, dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, a, b, out);
    FEM_HIP(hipGetLastError());
}

void launch_mask_copy(const fem_handle *h, const double *in, double *out, hipStream_t s) {
    if (h->g.N == 0) return;
    hipLaunchKernelGGL(k_mask_copy, dim3(grid_for(h->g.N, kThreads)), dim3(kThreads), 0, s, h->g.N, h->m.mask, in,
                       out);
    FEM_HIP(hipGetLastError());
}

void launch_sub(const double *a, const double *b, double *out, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_sub, dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, a, b, out);
    FEM_HIP(hipGetLastError());
}

void launch_export(const fem_handle *h, int64_t *row_ptr, int32_t *col_idx, int32_t *slot, int64_t *diag,
                   int32_t *tperm, hipStream_t s) {
    const Graph &g = h->g;
    if (row_ptr) FEM_HIP(hipMemcpyAsync(row_ptr, g.row_ptr, (g.N + 1) * sizeof(int64_t), hipMemcpyDeviceToDevice, s));
    const int nd = g.nd;
    if ((col_idx || tperm) && g.nnz > 0) {
        dim3 grid(grid_for(g.nnz, kThreads));
        if (nd == 1)
            hipLaunchKernelGGL(k_export_cols<1>, grid, dim3(kThreads), 0, s, g.nnzb, g.node_ptr, g.node_nb, g.blk_row,
                               g.mirror, g.row_ptr, col_idx, tperm);
        else
            hipLaunchKernelGGL(k_export_cols<3>, grid, dim3(kThreads), 0, s, g.nnzb, g.node_ptr, g.node_nb, g.blk_row,
                               g.mirror, g.row_ptr, col_idx, tperm);
    }
    if (slot && g.Ne > 0) {
        int64_t tot = g.Ne * 64 * nd * nd;
        dim3 grid(grid_for(tot, kThreads));
        if (nd == 1)
            hipLaunchKernelGGL(k_export_slots<1>, grid, dim3(kThreads), 0, s, g.Ne, h->m.conn, g.bslot, g.node_ptr,
                               g.row_ptr, slot);
        else
            hipLaunchKernelGGL(k_export_slots<3>, grid, dim3(kThreads), 0, s, g.Ne, h->m.conn, g.bslot, g.node_ptr,
                               g.row_ptr, slot);
    }
    if (diag && g.N > 0) {
        dim3 grid(grid_for(g.N, kThreads));
        if (nd == 1)
            hipLaunchKernelGGL(k_export_diag<1>, grid, dim3(kThreads), 0, s, g.N, g.bdiag, g.node_ptr, g.row_ptr, diag);
        else
            hipLaunchKernelGGL(k_export_diag<3>, grid, dim3(kThreads), 0, s, g.N, g.bdiag, g.node_ptr, g.row_ptr, diag);
    }
    FEM_HIP(hipGetLastError());
}

}  // namespace fem
