// Element-level kernels for HEX8 meshes on gfx950.
//
// Work mapping: one element per group of 8 consecutive lanes, lane a <-> local
// node a (so a 64-wide wavefront holds 8 elements and every cross-lane exchange
// stays inside a wavefront); per-point work is done once per Gauss point, lane q <->
// point q, and handed on through LDS.  The tangent's row blocks take two lanes per node
// (k_tangent_blocks).
//
// Element outputs go to a per-element scratch area and are summed per node / per
// CSR block by separate gather kernels: every global entry is written exactly once,
// with no atomics on values and a fixed summation order (deterministic).
//
// Paper: element residual R_e and K_e = dr_e/dU_e (Sec. 2.2), constitutive laws
// (Sec. 2.3, Eq. (linear_elasticity), Eq. (neo-hookean)), assembly (Alg. 1).
#include <algorithm>
#include <vector>

#include "internal.h"
#include "lanes.h"

namespace fem {

namespace {

constexpr int kThreads = 256;
constexpr int kElemsPerBlock = kThreads / 8;

__device__ __forceinline__ int ref_sign(int a, int j) {
    // reference coordinates of HEX8 node a: x = (a ^ (a >> 1)) & 1, y = (a >> 1) & 1, z = (a >> 2) & 1
    int bit = (j == 0) ? ((a ^ (a >> 1)) & 1) : (j == 1 ? ((a >> 1) & 1) : ((a >> 2) & 1));
    return bit ? 1 : -1;
}

// Sum over the 8 lanes of an element (DPP butterfly; every lane gets the total).
template <typename T>
__device__ __forceinline__ T sum8(T v) {
    return lane_sum8(v);
}

template <typename T>
__device__ __forceinline__ T det3(const T A[3][3]) {
    return A[0][0] * (A[1][1] * A[2][2] - A[1][2] * A[2][1]) - A[0][1] * (A[1][0] * A[2][2] - A[1][2] * A[2][0]) +
           A[0][2] * (A[1][0] * A[2][1] - A[1][1] * A[2][0]);
}

// B = A^{-T} (so that B g = A^{-T} g), given det(A) = d.
template <typename T>
__device__ __forceinline__ void inv_transpose3(const T A[3][3], T d, T B[3][3]) {
    T id = T(1) / d;
    B[0][0] = (A[1][1] * A[2][2] - A[1][2] * A[2][1]) * id;
    B[1][0] = (A[0][2] * A[2][1] - A[0][1] * A[2][2]) * id;
    B[2][0] = (A[0][1] * A[1][2] - A[0][2] * A[1][1]) * id;
    B[0][1] = (A[1][2] * A[2][0] - A[1][0] * A[2][2]) * id;
    B[1][1] = (A[0][0] * A[2][2] - A[0][2] * A[2][0]) * id;
    B[2][1] = (A[0][2] * A[1][0] - A[0][0] * A[1][2]) * id;
    B[0][2] = (A[1][0] * A[2][1] - A[1][1] * A[2][0]) * id;
    B[1][2] = (A[0][1] * A[2][0] - A[0][0] * A[2][1]) * id;
    B[2][2] = (A[0][0] * A[1][1] - A[0][1] * A[1][0]) * id;
}

__device__ __forceinline__ double modulus(const Material &m, double theta) {
    return m.pmap == FEM_THETA_SIMP ? m.simp_emin + pow(theta, m.simp_p) * (m.simp_e0 - m.simp_emin) : theta;
}

__device__ __forceinline__ double dmodulus(const Material &m, double theta) {
    return m.pmap == FEM_THETA_SIMP ? m.simp_p * pow(theta, m.simp_p - 1.0) * (m.simp_e0 - m.simp_emin) : 1.0;
}

// Per-lane geometry at Gauss point q: physical gradient g of this lane's shape
// function and the Jacobian determinant (identical in all 8 lanes).
template <typename T>
__device__ __forceinline__ T gp_geometry(int a, int q, const T X[3], T g[3]) {
    const T gq = T(0.57735026918962576451);  // 1/sqrt(3)
    T xi[3] = {(q & 1) ? gq : -gq, (q & 2) ? gq : -gq, (q & 4) ? gq : -gq};
    T l[3], s[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        s[j] = T(ref_sign(a, j));
        l[j] = T(0.5) * (T(1) + s[j] * xi[j]);
    }
    T dN[3] = {T(0.5) * s[0] * l[1] * l[2], T(0.5) * s[1] * l[0] * l[2], T(0.5) * s[2] * l[0] * l[1]};
    T J[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) J[i][j] = sum8(X[i] * dN[j]);
    T d = det3(J);
    T Bt[3][3];
    inv_transpose3(J, d, Bt);
#pragma unroll
    for (int i = 0; i < 3; ++i) g[i] = Bt[i][0] * dN[0] + Bt[i][1] * dN[1] + Bt[i][2] * dN[2];
    return d;
}

// Gradient of a nodal field (ND components) at the Gauss point: G[i][J] = sum_a U_a,i g_a,J.
template <int ND, typename T>
__device__ __forceinline__ void field_grad(const T U[ND], const T g[3], T G[3][3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) G[i][j] = (i < ND) ? sum8(U[i] * g[j]) : T(0);
}

// Neo-Hookean kinematic scalars at F = I + G.
template <typename T>
struct NHState {
    T F[3][3], H[3][3];  // H = F^{-T}
    T J, I1, c, alpha, beta, pcoef;
};

template <typename T>
__device__ __forceinline__ bool nh_state(const T G[3][3], T mod, T bulk_ratio, NHState<T> &s) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) s.F[i][j] = G[i][j] + (i == j ? T(1) : T(0));
    s.J = det3(s.F);
    bool ok = s.J > T(0);
    T J = ok ? s.J : T(1);
    inv_transpose3(s.F, J, s.H);
    T I1 = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) I1 += s.F[i][j] * s.F[i][j];
    s.I1 = I1;
    T kappa = bulk_ratio * mod;
    T cr = cbrt(J);
    s.c = mod / (cr * cr);  // G J^{-2/3}
    s.alpha = T(2.0 / 9.0) * s.c * I1 + kappa * (T(2) * J * J - J);
    s.beta = s.c * I1 * T(1.0 / 3.0) - kappa * (J * J - J);
    s.pcoef = kappa * J * (J - T(1)) - s.c * I1 * T(1.0 / 3.0);  // P g = c F g + pcoef H g
    return ok;
}

template <typename T>
__device__ __forceinline__ void matvec3(const T A[3][3], const T x[3], T y[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) y[i] = A[i][0] * x[0] + A[i][1] * x[1] + A[i][2] * x[2];
}

// Perfect J2 plasticity at one Gauss point (Sec. 2.3, plasticity paragraph).  hq holds
// the committed state of the point: total strain then stress, each as (xx, yy, zz, yz,
// xz, xy).  Trial stress from the strain increment sym(G) - eps, deviator s and
// s_vm = sqrt(3/2 s:s); above the yield stress the deviator is scaled back onto the
// surface (radial return).  The consistent tangent of that map, d sigma / d grad u
// (hand-derived; the paper leaves it to automatic differentiation), is
//   A = lw I(x)I + mup (delta_ik delta_jl + delta_il delta_jk) - beta s(x)s
// with kappa = lambda + 2 mu / 3; elastic: mup = mu, beta = 0; plastic:
// mup = mu sigma_y / s_vm, beta = 3 mup / s_vm^2; and lw = kappa - 2 mup / 3.
template <typename T>
struct J2State {
    T sig[6], dev[6];  // returned stress and trial deviator, (xx, yy, zz, yz, xz, xy)
    T lw, mup, beta;
};

template <typename T>
__device__ __forceinline__ void j2_state(const Material &m, T E, const T G[3][3], const double *hq, J2State<T> &s) {
    const T nu = T(m.nu);
    const T lam = E * nu / ((T(1) + nu) * (T(1) - T(2) * nu)), mu = E / (T(2) * (T(1) + nu));
    T de[6] = {G[0][0], G[1][1], G[2][2], T(0.5) * (G[1][2] + G[2][1]), T(0.5) * (G[0][2] + G[2][0]),
               T(0.5) * (G[0][1] + G[1][0])};
#pragma unroll
    for (int c = 0; c < 6; ++c) de[c] -= T(hq[c]);
    const T tr = de[0] + de[1] + de[2];
    T st[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) st[c] = T(hq[6 + c]) + T(2) * mu * de[c] + (c < 3 ? lam * tr : T(0));
    const T p = (st[0] + st[1] + st[2]) * T(1.0 / 3.0);
    T ss = T(0);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        s.dev[c] = st[c] - (c < 3 ? p : T(0));
        ss += (c < 3 ? T(1) : T(2)) * s.dev[c] * s.dev[c];
    }
    const T svm = sqrt(T(1.5) * ss), f = svm - T(m.yield_stress);
    const bool plastic = f > T(0);
    const T kappa = lam + T(2.0 / 3.0) * mu;
    s.mup = plastic ? mu * T(m.yield_stress) / svm : mu;
    s.beta = plastic ? T(3) * s.mup / (svm * svm) : T(0);
    s.lw = kappa - T(2.0 / 3.0) * s.mup;
#pragma unroll
    for (int c = 0; c < 6; ++c) s.sig[c] = plastic ? st[c] - s.dev[c] / svm * f : st[c];
}

// y = S x for a symmetric tensor stored as (xx, yy, zz, yz, xz, xy).
template <typename T>
__device__ __forceinline__ void symvec(const T S[6], const T x[3], T y[3]) {
    y[0] = S[0] * x[0] + S[5] * x[1] + S[4] * x[2];
    y[1] = S[5] * x[0] + S[1] * x[1] + S[3] * x[2];
    y[2] = S[4] * x[0] + S[3] * x[1] + S[2] * x[2];
}

// Flux applied to this lane's shape gradient: out = f(G) g (the integrand of R_e
// at one Gauss point, before the quadrature weight).  Returns false if det F <= 0.
// hq: the Gauss point's committed J2 state (unused by the other laws).
// First Piola flux P(G) as a 3x3 matrix (rows >= ND are zero): the element residual
// of node a is sum_q detJ P g_a.
template <int MODEL, typename T>
__device__ __forceinline__ bool flux_mat(const Material &m, T mod, const T G[3][3], T P[3][3], const double *hq) {
    if constexpr (MODEL == FEM_POISSON) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) P[i][j] = (i == 0) ? mod * G[0][j] : T(0);
        return true;
    } else if constexpr (MODEL == FEM_LINEAR_ELASTIC) {
        T nu = T(m.nu);
        T lam = mod * nu / ((T(1) + nu) * (T(1) - T(2) * nu)), mu = mod / (T(2) * (T(1) + nu));
        T tr = G[0][0] + G[1][1] + G[2][2];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) P[i][j] = mu * (G[i][j] + G[j][i]) + (i == j ? lam * tr : T(0));
        return true;
    } else {
        static_assert(MODEL == FEM_NEO_HOOKEAN, "the J2 law uses j2_flux_dot");
        NHState<T> s;
        bool ok = nh_state(G, mod, T(m.bulk_ratio), s);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) P[i][j] = s.c * s.F[i][j] + s.pcoef * s.H[i][j];
        return ok;
    }
}

// Directional derivative of the flux, dP = A(G) : dG, as a 3x3 matrix.
template <int MODEL, typename T>
__device__ __forceinline__ bool dflux_mat(const Material &m, T mod, const T G[3][3], const T dG[3][3], T dP[3][3],
                                          const double *hq) {
    if constexpr (MODEL == FEM_POISSON || MODEL == FEM_LINEAR_ELASTIC) {
        return flux_mat<MODEL, T>(m, mod, dG, dP, hq);  // linear laws
    } else {
        static_assert(MODEL == FEM_NEO_HOOKEAN, "the J2 law uses j2_dflux_dot");
        NHState<T> s;
        bool ok = nh_state(G, mod, T(m.bulk_ratio), s);
        T HdF = T(0), FdF = T(0);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                HdF += s.H[i][j] * dG[i][j];
                FdF += s.F[i][j] * dG[i][j];
            }
        // dF^T H, then H (dF^T H)
        T DH[3][3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) DH[k][j] = dG[0][k] * s.H[0][j] + dG[1][k] * s.H[1][j] + dG[2][k] * s.H[2][j];
        T c23 = T(2.0 / 3.0) * s.c;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const T HDH = s.H[i][0] * DH[0][j] + s.H[i][1] * DH[1][j] + s.H[i][2] * DH[2][j];
                dP[i][j] = s.c * dG[i][j] - c23 * (s.F[i][j] * HdF + s.H[i][j] * FdF) + s.alpha * s.H[i][j] * HdF +
                           s.beta * HDH;
            }
        return ok;
    }
}

// J2 flux and its derivative applied to this lane's gradient g (the per-lane form used
// by the J2 vector kernel): out = sigma g, and out = (A : dG) g.
template <typename T>
__device__ __forceinline__ void j2_flux_dot(const Material &m, T mod, const T G[3][3], const T g[3], T out[3],
                                            const double *hq) {
    J2State<T> s;
    j2_state(m, mod, G, hq, s);
    symvec(s.sig, g, out);
}

template <typename T>
__device__ __forceinline__ void j2_dflux_dot(const Material &m, T mod, const T G[3][3], const T dG[3][3],
                                             const T g[3], T out[3], const double *hq) {
    J2State<T> s;
    j2_state(m, mod, G, hq, s);
    const T tr = dG[0][0] + dG[1][1] + dG[2][2];
    const T sd = s.dev[0] * dG[0][0] + s.dev[1] * dG[1][1] + s.dev[2] * dG[2][2] + s.dev[3] * (dG[1][2] + dG[2][1]) +
                 s.dev[4] * (dG[0][2] + dG[2][0]) + s.dev[5] * (dG[0][1] + dG[1][0]);
    T sg[3];
    symvec(s.dev, g, sg);
#pragma unroll
    for (int i = 0; i < 3; ++i)
        out[i] = s.lw * tr * g[i] +
                 s.mup * ((dG[i][0] + dG[0][i]) * g[0] + (dG[i][1] + dG[1][i]) * g[1] + (dG[i][2] + dG[2][i]) * g[2]) -
                 s.beta * sd * sg[i];
}

// Reference gradients dN_b(xi_q) of the 8 shape functions at Gauss point q.
template <typename T>
__device__ __forceinline__ void ref_grad(int b, int q, T dN[3]) {
    const T gq = T(0.57735026918962576451);  // 1/sqrt(3)
    T l[3], sg[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const T xi = ((q >> j) & 1) ? gq : -gq;
        sg[j] = T(ref_sign(b, j));
        l[j] = T(0.5) * (T(1) + sg[j] * xi);
    }
    dN[0] = T(0.5) * sg[0] * l[1] * l[2];
    dN[1] = T(0.5) * sg[1] * l[0] * l[2];
    dN[2] = T(0.5) * sg[2] * l[0] * l[1];
}

struct ElemIds {
    int64_t e;
    int a, el;
    bool valid;
};

__device__ __forceinline__ ElemIds elem_ids(int64_t Ne) {
    ElemIds id;
    id.a = threadIdx.x & 7;
    id.el = threadIdx.x >> 3;
    int64_t e = int64_t(blockIdx.x) * kElemsPerBlock + id.el;
    id.valid = e < Ne;
    id.e = id.valid ? e : Ne - 1;  // idle groups recompute the last element and store nothing
    return id;
}

// Loads this lane's node.  Coordinates (and, with rel_u, the field) are taken
// relative to local node 0 of the element, in FP64 before rounding to T: the
// gradients are unchanged (the shape-function gradients sum to zero) but the
// differences of nearby absolute values no longer cancel in T arithmetic.
// All loads go out before the first is used; what is read is fixed at compile time (a test
// of the pointers between the loads made every component wait for the one before it).
enum : int { LOAD_COORDS = 0, LOAD_FIELD = 1, LOAD_REL = 2, LOAD_MASKED = 4 };  // the field; minus node 0's; 0 where masked
template <int ND, int FLAGS, typename T>
__device__ __forceinline__ void load_node(const double *coords, const int32_t *conn, const double *u,
                                          const uint8_t *mask, const ElemIds &id, T X[3], T U[ND]) {
    constexpr bool kField = FLAGS & LOAD_FIELD, kRel = FLAGS & LOAD_REL, kMask = FLAGS & LOAD_MASKED;
    const int64_t n = conn[id.e * 8 + id.a];
    const int64_t n0 = conn[id.e * 8];
    double x[3], x0[3], v[ND], v0[ND];
    uint8_t m[ND], m0[ND];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        x[i] = coords[3 * n + i];
        x0[i] = coords[3 * n0 + i];
    }
#pragma unroll
    for (int i = 0; i < ND; ++i) {
        v[i] = kField ? u[ND * n + i] : 0.0;
        v0[i] = kField && kRel ? u[ND * n0 + i] : 0.0;
        m[i] = kMask ? mask[ND * n + i] : 0;
        m0[i] = kMask && kRel ? mask[ND * n0 + i] : 0;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) X[i] = T(x[i] - x0[i]);
#pragma unroll
    for (int i = 0; i < ND; ++i) U[i] = T((m[i] ? 0.0 : v[i]) - (m0[i] ? 0.0 : v0[i]));
}

// Exchanges along the edges of the reference cube (see k_element_vec): the weights of the
// near and the far node of a point in one direction are p = (1 + g) / 2 and p r.
constexpr double kFar = 0.26794919243112270647;  // r = (1 - g) / (1 + g) = 2 - sqrt(3), g = 1 / sqrt(3)
// (p^2 / 2)^3, p^2 = (2 + sqrt(3)) / 6: the factors left out of the determinant
constexpr double kCornerDet = 0.03008145955644280059;
// (lp^2 / 2) (2 / p^2)^2 = 2 / p^2 with lp = p: the rule's weight of a point of the tangent
constexpr double kPointWeight = 3.21539030917347247767;

// Derivatives along the three directions at this lane's point of the field with value v at
// this lane's node, without their factors s_k p^2 / 2.
__device__ __forceinline__ void corner_grad(double v, double g[3]) {
    const double v0 = dpp_read<kDppXor1>(v);
    const double d0 = v - v0, i0 = fma(kFar, v0, v);
    const double d01 = fma(kFar, dpp_read<kDppXor2>(d0), d0);
    const double i0x = dpp_read<kDppXor2>(i0);
    const double d1 = i0 - i0x, i1 = fma(kFar, i0x, i0);
    g[0] = fma(kFar, dpp_read<kDppHalfMirror>(d01), d01);
    g[1] = fma(kFar, dpp_read<kDppHalfMirror>(d1), d1);
    g[2] = i1 - dpp_read<kDppHalfMirror>(i1);
}

// The transpose: the sum over the points of M[k] times the derivative of this lane's node's shape
// function in direction k, M with the factors left out above.
__device__ __forceinline__ double corner_div(const double M[3]) {
    double a = M[0] - dpp_read<kDppXor1>(M[0]);
    double b = fma(kFar, dpp_read<kDppXor1>(M[1]), M[1]);
    double c = fma(kFar, dpp_read<kDppXor1>(M[2]), M[2]);
    a = fma(kFar, dpp_read<kDppXor2>(a), a);
    b -= dpp_read<kDppXor2>(b);
    c = fma(kFar, dpp_read<kDppXor2>(c), c);
    const double ab = a + b;
    return ab + c + dpp_read<kDppHalfMirror>(fma(kFar, ab, -c));
}

// ------------------------------------------------------------------ residual-type kernels
enum { VEC_RESIDUAL = 0, VEC_JVP = 1, VEC_VJP = 2, VEC_LIFT = 3, VEC_MASS = 4 };

// (slot s = kpos[e*8 + a]: node-major incidence order, so each node's terms are contiguous)
// VEC_RESIDUAL: scratch[s][i] = sum_q detJ f(grad u) g_a            (modulus m(theta_e))
// VEC_JVP:      scratch[s][i] = sum_q detJ (A(grad u) : grad v) g_a  (v with Dirichlet dofs zeroed)
// VEC_VJP:      g[e] = -m'(theta_e) sum_{a,i free} lam_a,i sum_q detJ f_unit(grad u) g_a
// VEC_LIFT:     as VEC_JVP but with v used on every dof (v is nonzero on Dirichlet dofs only)
//
// 8 lanes per element, no LDS.  A lane is one corner (s0, s1, s2) of the reference cube: the
// element's node there and the Gauss point nearest to it.  In each direction the two nodes
// enter a point with the weights p (1 + g) / 2 and p r, and a point enters its two nodes with
// the same, so gradients at the points and sums over the points are three exchanges along
// the cube's edges, each a register move and one multiply-add (corner_grad, corner_div).  A
// gradient costs 6 exchanges and 8 operations per value instead of 24 multiply-adds and
// the shape-function products; the Jacobian inverse and the constitutive update are done
// once per point.  What bounds it is FP64 arithmetic and the moves.  Neo-Hookean residual, 100^3
// elements: 229 -> 176 us; product with the tangent and VJP, 64^3: 123 -> 95 us together
// (before: node values through LDS and the shape functions of every node at every point).
template <int MODEL, int ND, int MODE>
__global__ __launch_bounds__(kThreads) void k_element_vec(int64_t Ne, const double *__restrict__ coords,
                                                          const int32_t *__restrict__ conn,
                                                          const int32_t *__restrict__ kpos,
                                                          const uint8_t *__restrict__ mask, Material mat,
                                                          const double *__restrict__ theta,
                                                          const double *__restrict__ u,
                                                          const double *__restrict__ v,
                                                          const double *__restrict__ hist, double *__restrict__ out,
                                                          int *status) {
    constexpr bool kDir = MODE == VEC_JVP || MODE == VEC_LIFT;
    if constexpr (MODEL == FEM_J2_PLASTIC) {
        // J2 keeps the per-lane form (every lane walks the 8 points for its own node): the
        // loading-unloading path near the limit load has a nearly singular tangent, and
        // its Newton iterations were measured to converge with this form's rounding.
        ElemIds id = elem_ids(Ne);
        double X[3], U[ND], W[ND];
        load_node<ND, LOAD_FIELD | LOAD_REL>(coords, conn, u, nullptr, id, X, U);
        if (MODE != VEC_RESIDUAL)
            load_node<ND, LOAD_FIELD | (MODE == VEC_LIFT ? 0 : LOAD_MASKED) | (MODE != VEC_VJP ? LOAD_REL : 0)>(
                coords, conn, v, mask, id, X, W);
        double th = theta[id.e];
        double mod = (MODE == VEC_VJP) ? 1.0 : modulus(mat, th);
        double acc[3] = {0, 0, 0};
        bool mesh_ok = true;
#pragma unroll 1
        for (int q = 0; q < 8; ++q) {
            double g[3];
            double dJ = gp_geometry(id.a, q, X, g);
            mesh_ok &= dJ > 0.0;
            double G[3][3], o[3];
            field_grad<ND>(U, g, G);
            const double *hq = hist + (id.e * 8 + q) * 12;
            if (kDir) {
                double dG[3][3];
                field_grad<ND>(W, g, dG);
                j2_dflux_dot<double>(mat, mod, G, dG, g, o, hq);
            } else {
                j2_flux_dot<double>(mat, mod, G, g, o, hq);
            }
#pragma unroll
            for (int i = 0; i < ND; ++i) acc[i] += dJ * o[i];
        }
        if (id.valid && id.a == 0 && !mesh_ok) atomicOr(status, ST_MESH);
        if (MODE == VEC_VJP) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < ND; ++i) s += W[i] * acc[i];
            s = sum8(s);
            if (id.valid && id.a == 0) out[id.e] = -dmodulus(mat, th) * s;
        } else if (id.valid) {
#pragma unroll
            for (int i = 0; i < ND; ++i) out[int64_t(kpos[id.e * 8 + id.a]) * ND + i] = acc[i];
        }
    } else {
        ElemIds id = elem_ids(Ne);
        // corner of this lane: bits of c.  A step along direction 0 is lane ^ 1, along direction
        // 1 lane ^ 2 and along direction 2 lane ^ 7 (each one DPP move).
        const int c = id.a ^ ((id.a & 4) ? 3 : 0);
        id.a = c ^ ((c >> 1) & 1);  // local node there
        double X[3], U[ND], W[ND];
        load_node<ND, LOAD_FIELD | LOAD_REL>(coords, conn, u, nullptr, id, X, U);
        if (MODE != VEC_RESIDUAL)
            load_node<ND, LOAD_FIELD | (MODE == VEC_LIFT ? 0 : LOAD_MASKED) | (MODE != VEC_VJP ? LOAD_REL : 0)>(
                    coords, conn, v, mask, id, X, W);
        const double th = theta[id.e];
        const double mod = (MODE == VEC_VJP) ? 1.0 : modulus(mat, th);
        // J and the gradients come without the factor p^2 / 2 of every column and the sign s_k of
        // column k: they cancel in G = Gr J^{-1} and, up to the signs of the sums' differences, in
        // d P J^{-T} dN; only the determinant needs them.
        double J[3][3], Gr[3][3] = {}, Wr[3][3] = {};
#pragma unroll
        for (int i = 0; i < 3; ++i) corner_grad(X[i], J[i]);
#pragma unroll
        for (int i = 0; i < ND; ++i) corner_grad(U[i], Gr[i]);
        if constexpr (kDir)
#pragma unroll
            for (int i = 0; i < ND; ++i) corner_grad(W[i], Wr[i]);
        const double dj = det3(J);
        const double d = (__popc(c) & 1) ? kCornerDet * dj : -kCornerDet * dj;
        const bool mesh_ok = d > 0.0;
        double Bt[3][3];
        inv_transpose3(J, dj, Bt);
        double G[3][3], dG[3][3], P[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                G[i][j] = Gr[i][0] * Bt[j][0] + Gr[i][1] * Bt[j][1] + Gr[i][2] * Bt[j][2];
                dG[i][j] = Wr[i][0] * Bt[j][0] + Wr[i][1] * Bt[j][1] + Wr[i][2] * Bt[j][2];
            }
        bool mat_ok;
        if constexpr (kDir) mat_ok = dflux_mat<MODEL, double>(mat, mod, G, dG, P, nullptr);
        else mat_ok = flux_mat<MODEL, double>(mat, mod, G, P, nullptr);
        double acc[ND];
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            double M[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) M[k] = d * (P[i][0] * Bt[0][k] + P[i][1] * Bt[1][k] + P[i][2] * Bt[2][k]);
            acc[i] = corner_div(M);
        }
        if (id.valid && (!mesh_ok || !mat_ok))
            atomicOr(status, (!mesh_ok ? ST_MESH : 0) | (!mat_ok ? ST_INVERTED : 0));
        if (MODE == VEC_VJP) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < ND; ++i) s += W[i] * acc[i];
            s = sum8(s);
            if (id.valid && id.a == 0) out[id.e] = -dmodulus(mat, th) * s;
        } else if (id.valid) {
#pragma unroll
            for (int i = 0; i < ND; ++i) out[int64_t(kpos[id.e * 8 + id.a]) * ND + i] = acc[i];
        }
    }
}

// Consistent mass product: scratch[s][i] = sum_q detJ N_a(xi_q) sum_b N_b(xi_q) x_b,i
// (the load of a nodal field x interpolated with the shape functions; Sec. 2.1,
// the body-force term of Eq. (weak)).
template <int ND>
__global__ __launch_bounds__(kThreads) void k_element_mass(int64_t Ne, const double *__restrict__ coords,
                                                           const int32_t *__restrict__ conn,
                                                           const int32_t *__restrict__ kpos,
                                                           const double *__restrict__ x, double *__restrict__ out,
                                                           int *status) {
    ElemIds id = elem_ids(Ne);
    double X[3], Xv[ND];
    load_node<ND, LOAD_FIELD>(coords, conn, x, nullptr, id, X, Xv);
    const double gq = 0.57735026918962576451;
    double acc[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) acc[i] = 0.0;
    bool mesh_ok = true;
#pragma unroll 1
    for (int q = 0; q < 8; ++q) {
        double g[3];
        const double dJ = gp_geometry(id.a, q, X, g);
        mesh_ok &= dJ > 0.0;
        double Na = 1.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double xi = (q >> j) & 1 ? gq : -gq;
            Na *= 0.5 * (1.0 + double(ref_sign(id.a, j)) * xi);
        }
#pragma unroll
        for (int i = 0; i < ND; ++i) acc[i] += dJ * Na * sum8(Na * Xv[i]);
    }
    if (id.valid && id.a == 0 && !mesh_ok) atomicOr(status, ST_MESH);
    if (id.valid)
#pragma unroll
        for (int i = 0; i < ND; ++i) out[int64_t(kpos[id.e * 8 + id.a]) * ND + i] = acc[i];
}

// J2 history commit after a converged load step: lane a updates Gauss point a of its
// element, eps <- sym(grad u) and sigma <- the returned stress of j2_state.  Each
// point reads and then writes only its own record, so the update is in place.
__global__ __launch_bounds__(kThreads) void k_j2_commit(int64_t Ne, const double *__restrict__ coords,
                                                       const int32_t *__restrict__ conn, Material mat,
                                                       const double *__restrict__ theta,
                                                       const double *__restrict__ u, double *__restrict__ hist) {
    ElemIds id = elem_ids(Ne);
    double X[3], U[3];
    load_node<3, LOAD_FIELD | LOAD_REL>(coords, conn, u, nullptr, id, X, U);
    double Gm[3][3] = {};
#pragma unroll 1
    for (int q = 0; q < 8; ++q) {
        double g[3], G[3][3];
        gp_geometry(id.a, q, X, g);
        field_grad<3>(U, g, G);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) Gm[i][j] = (q == id.a) ? G[i][j] : Gm[i][j];
    }
    if (!id.valid) return;
    double *hq = hist + (id.e * 8 + id.a) * 12;
    J2State<double> st;
    j2_state(mat, modulus(mat, theta[id.e]), Gm, hq, st);
    const double eps[6] = {Gm[0][0], Gm[1][1], Gm[2][2], 0.5 * (Gm[1][2] + Gm[2][1]), 0.5 * (Gm[0][2] + Gm[2][0]),
                           0.5 * (Gm[0][1] + Gm[1][0])};
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        hq[c] = eps[c];
        hq[6 + c] = st.sig[c];
    }
}

// Per-block partial sums of sum_q detJ sigma_q (6 components) and sum_q detJ over the
// committed J2 history: lane a takes Gauss point a; partials[block * 7 + c].
__global__ __launch_bounds__(kThreads) void k_j2_average(int64_t Ne, const double *__restrict__ coords,
                                                        const int32_t *__restrict__ conn,
                                                        const double *__restrict__ hist, double *partials) {
    __shared__ double red[kThreads / 64][7];
    ElemIds id = elem_ids(Ne);
    double X[3], U[1];
    load_node<1, LOAD_COORDS>(coords, conn, nullptr, nullptr, id, X, U);
    double w = 0.0;
#pragma unroll 1
    for (int q = 0; q < 8; ++q) {
        double g[3];
        const double dJ = gp_geometry(id.a, q, X, g);
        w = (q == id.a) ? dJ : w;
    }
    if (!id.valid) w = 0.0;
    const double *hs = hist + (id.e * 8 + id.a) * 12 + 6;
    double v[7];
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] = w * hs[c];
    v[6] = w;
#pragma unroll
    for (int c = 0; c < 7; ++c) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[c] += __shfl_xor(v[c], o, 64);
    }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int c = 0; c < 7; ++c) red[threadIdx.x >> 6][c] = v[c];
    __syncthreads();
    if (threadIdx.x < 7) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kThreads / 64; ++k) t += red[k][threadIdx.x];
        partials[int64_t(blockIdx.x) * 7 + threadIdx.x] = t;
    }
}

// Sum element contributions per dof, eight lanes per node, one of its slots each: the slots of
// consecutive nodes are one run of memory, read once.  What bounds it is that run: 64^3
// elements, 60 MB, 18.8 -> 11.7 us; 100^3, 240 MB, 73 -> 53 us (a thread per dof walked its
// node's slots at a stride).
// VEC_RESIDUAL: out[d] = sum - lf * F[d], 0 on Dirichlet dofs.
// VEC_JVP:      out[d] = sum, v[d] on Dirichlet dofs.
// VEC_LIFT:     out[d] = sum, 0 on Dirichlet dofs.
template <int ND, int MODE>
__global__ __launch_bounds__(256) void k_gather_vec(int64_t Nn, const int64_t *__restrict__ ne_ptr,
                                                    const double *__restrict__ scratch,
                                                    const uint8_t *__restrict__ mask, const double *__restrict__ F,
                                                    double lf, const double *__restrict__ v,
                                                    double *__restrict__ out, int *status) {
    const int l8 = threadIdx.x & 7;
    const int64_t n = int64_t(blockIdx.x) * (blockDim.x / 8) + threadIdx.x / 8;
    const bool live = n < Nn;  // (every lane stays active for the sums)
    const int64_t k0 = live ? ne_ptr[n] : 0, k1 = live ? ne_ptr[n + 1] : 0;
    const bool own = live && l8 < ND;
    const int64_t d = ND * n + l8;
    const bool fixed = own && mask && mask[d];
    const double f = own && MODE == VEC_RESIDUAL ? F[d] : 0.0;
    double s[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) s[i] = 0.0;
    for (int64_t k = k0 + l8; k < k1; k += 8)
#pragma unroll
        for (int i = 0; i < ND; ++i) s[i] += scratch[k * ND + i];
#pragma unroll
    for (int i = 0; i < ND; ++i) s[i] = sum8(s[i]);
    if (!own) return;
    double sum = s[0];
    if constexpr (ND == 3) sum = l8 == 1 ? s[1] : (l8 == 2 ? s[2] : s[0]);
    double r;
    if (fixed) r = (MODE == VEC_JVP) ? v[d] : 0.0;
    else r = (MODE == VEC_RESIDUAL) ? sum - lf * f : sum;
    if (!isfinite(r)) atomicOr(status, ST_NAN);
    out[d] = r;
}

// ------------------------------------------------------------------ tangent kernel
// Lane a accumulates the row block K_e[(a,i), (b,k)] for all b, i, k and writes it to
// scratch[((kpos[e*8 + a])*8 + b)*ND*ND + i*ND + k]: the row blocks feeding node
// conn[e][a] are contiguous, so the gather reads each node's 8 row blocks as one run.
template <int MODEL, int ND, typename T>
__global__ __launch_bounds__(kThreads, sizeof(T) == 4 ? 3 : 2) void k_element_tangent(int64_t Ne, const double *__restrict__ coords,
                                                              const int32_t *__restrict__ conn,
                                                              const int32_t *__restrict__ kpos, Material mat,
                                                              const double *__restrict__ theta,
                                                              const double *__restrict__ u,
                                                              const double *__restrict__ hist, T *__restrict__ ke,
                                                              int *status) {
    // per-node data shared through LDS: g (all laws), F g and F^{-T} g (neo-Hookean),
    // s g with the trial deviator s (J2)
    constexpr int NV = (MODEL == FEM_NEO_HOOKEAN) ? 9 : (MODEL == FEM_J2_PLASTIC ? 6 : 3);
    constexpr int ES = 8 * NV + 1;  // padded element stride (bank spread)
    constexpr bool kNonlinear = MODEL == FEM_NEO_HOOKEAN || MODEL == FEM_J2_PLASTIC;
    __shared__ T lds[kElemsPerBlock * ES];
    ElemIds id = elem_ids(Ne);
    T X[3], U[ND];
    load_node<ND, kNonlinear ? LOAD_FIELD | LOAD_REL : LOAD_COORDS>(coords, conn, u, nullptr, id, X, U);
    T mod = T(modulus(mat, theta[id.e]));
    T K[8][ND][ND];
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
        for (int i = 0; i < ND; ++i)
#pragma unroll
            for (int k = 0; k < ND; ++k) K[b][i][k] = T(0);
    bool mesh_ok = true, mat_ok = true;
    T *my = lds + id.el * ES + id.a * NV;
    const T *el = lds + id.el * ES;
#pragma unroll 1
    for (int q = 0; q < 8; ++q) {
        T g[3];
        T dJ = gp_geometry(id.a, q, X, g);
        mesh_ok &= dJ > T(0);
        if constexpr (MODEL == FEM_NEO_HOOKEAN) {
            T G[3][3];
            field_grad<ND>(U, g, G);
            NHState<T> s;
            mat_ok &= nh_state(G, mod, T(mat.bulk_ratio), s);
            T f[3], h[3];
            matvec3(s.F, g, f);
            matvec3(s.H, g, h);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                my[i] = g[i];
                my[3 + i] = f[i];
                my[6 + i] = h[i];
            }
            __syncthreads();
            T cw = dJ * s.c, c23 = T(2.0 / 3.0) * cw, aw = dJ * s.alpha, bw = dJ * s.beta;
            // block (a, b): aw h_i hb_k + bw hb_i h_k - c23 (f_i hb_k + h_i fb_k) + delta_ik cw g.gb,
            // grouped by the factors of this node so each entry takes three FMAs
            T P[3], Q[3], R[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                P[i] = aw * h[i] - c23 * f[i];
                Q[i] = bw * h[i];
                R[i] = -c23 * h[i];
            }
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const T *o = el + b * NV;
                T gb[3] = {o[0], o[1], o[2]}, fb[3] = {o[3], o[4], o[5]}, hb[3] = {o[6], o[7], o[8]};
                T sdot = cw * (g[0] * gb[0] + g[1] * gb[1] + g[2] * gb[2]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        T v = fma(P[i], hb[k], K[b][i][k]);
                        v = fma(hb[i], Q[k], v);
                        v = fma(R[i], fb[k], v);
                        if (i == k) v += sdot;
                        K[b][i][k] = v;
                    }
            }
            __syncthreads();
        } else if constexpr (MODEL == FEM_J2_PLASTIC) {
            T G[3][3];
            field_grad<ND>(U, g, G);
            J2State<T> s;
            j2_state(mat, mod, G, hist + (id.e * 8 + q) * 12, s);
            T sg[3];
            symvec(s.dev, g, sg);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                my[i] = g[i];
                my[3 + i] = sg[i];
            }
            __syncthreads();
            T lw = dJ * s.lw, mw = dJ * s.mup, bw = dJ * s.beta;
            // block (a, b): lw g_i gb_k + mw g_k gb_i - bw sg_i sb_k + delta_ik mw g.gb, three FMAs
            // per entry with this node's factors taken first
            T P[3], Q[3], R[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                P[i] = lw * g[i];
                Q[i] = mw * g[i];
                R[i] = -bw * sg[i];
            }
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const T *o = el + b * NV;
                T gb[3] = {o[0], o[1], o[2]}, sb[3] = {o[3], o[4], o[5]};
                T sdot = mw * (g[0] * gb[0] + g[1] * gb[1] + g[2] * gb[2]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        T v = fma(P[i], gb[k], K[b][i][k]);
                        v = fma(gb[i], Q[k], v);
                        v = fma(R[i], sb[k], v);
                        if (i == k) v += sdot;
                        K[b][i][k] = v;
                    }
            }
            __syncthreads();
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) my[i] = g[i];
            __syncthreads();
            if constexpr (MODEL == FEM_LINEAR_ELASTIC) {
                T nu = T(mat.nu);
                T lw = dJ * mod * nu / ((T(1) + nu) * (T(1) - T(2) * nu)), mw = dJ * mod / (T(2) * (T(1) + nu));
                T P[3], Q[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    P[i] = lw * g[i];
                    Q[i] = mw * g[i];
                }
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const T *o = el + b * NV;
                    T gb[3] = {o[0], o[1], o[2]};
                    T sdot = mw * (g[0] * gb[0] + g[1] * gb[1] + g[2] * gb[2]);
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            // lw g_i gb_k + mw g_k gb_i + delta_ik mw g.gb
                            T v = fma(P[i], gb[k], K[b][i][k]);
                            v = fma(gb[i], Q[k], v);
                            if (i == k) v += sdot;
                            K[b][i][k] = v;
                        }
                }
            } else {
                T w = dJ * mod;
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const T *o = el + b * NV;
                    K[b][0][0] += w * (g[0] * o[0] + g[1] * o[1] + g[2] * o[2]);
                }
            }
            __syncthreads();
        }
    }
    if (id.valid && id.a == 0 && (!mesh_ok || !mat_ok))
        atomicOr(status, (!mesh_ok ? ST_MESH : 0) | (!mat_ok ? ST_INVERTED : 0));
    if (id.valid) {
        T *dst = ke + int64_t(kpos[id.e * 8 + id.a]) * 8 * ND * ND;
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int k = 0; k < ND; ++k) dst[(b * ND + i) * ND + k] = K[b][i][k];
    }
}

// Tangent values from element blocks: thread (block kb, row component i) sums the
// contributing element blocks of node-graph block kb = (n, j-th neighbour m) in
// element order, applies the symmetric Dirichlet elimination and writes row i of
// the block once:
//   LAYOUT_CSR: values[row_ptr[ND*n+i] + ND*j + k], k < ND;
//   LAYOUT_SYM: only blocks with m >= n, block-major at values[ND*ND*(up_base[n] +
//               kb - bdiag[n]) + ND*i + k] (the lower blocks are their transposes).
template <int ND, int LAYOUT, typename T>
__global__ __launch_bounds__(256) void k_gather_values(int64_t nnzb, const int64_t *__restrict__ node_ptr,
                                                       const int32_t *__restrict__ node_nb,
                                                       const int32_t *__restrict__ blk_row,
                                                       const int64_t *__restrict__ blk_ptr,
                                                       const int32_t *__restrict__ blk_src,
                                                       const int64_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ bdiag,
                                                       const int64_t *__restrict__ up_base,
                                                       const uint8_t *__restrict__ mask, const T *__restrict__ ke,
                                                       T *__restrict__ values, int *status) {
    int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= nnzb * ND) return;
    int64_t kb = t / ND;
    int i = int(t - kb * ND);
    int64_t n = blk_row[kb];
    int64_t m = node_nb[kb];
    if (LAYOUT == LAYOUT_SYM && m < n) return;
    T acc[ND];
#pragma unroll
    for (int k = 0; k < ND; ++k) acc[k] = T(0);
    for (int64_t s = blk_ptr[kb]; s < blk_ptr[kb + 1]; ++s) {
        const T *src = ke + int64_t(blk_src[s]) * ND * ND + i * ND;
#pragma unroll
        for (int k = 0; k < ND; ++k) acc[k] += src[k];
    }
    int64_t row = ND * n + i;
    bool bad = false;
    T *dst = (LAYOUT == LAYOUT_SYM) ? values + ND * ND * (up_base[n] + kb - bdiag[n]) + ND * i
                                    : values + row_ptr[row] + ND * (kb - node_ptr[n]);
#pragma unroll
    for (int k = 0; k < ND; ++k) {
        int64_t col = ND * m + k;
        T v = acc[k];
        if (mask && (mask[row] || mask[col])) v = (row == col) ? T(1) : T(0);
        bad |= !isfinite(v);
        dst[k] = v;
    }
    if (bad) atomicOr(status, ST_NAN);
}

// Inverse of an ND x ND block (FP64 cofactors), written row-major to out; false when
// the block is singular or not finite.
template <int ND, typename T>
__device__ __forceinline__ bool invert_block(const double B[ND][ND], T *out) {
    if constexpr (ND == 1) {
        out[0] = T(1.0 / B[0][0]);
        return B[0][0] != 0.0 && isfinite(B[0][0]);
    } else {
        const double d = det3(B);
        double C[3][3];
        inv_transpose3(B, d, C);  // C = B^{-T}
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c) out[i * 3 + c] = T(C[c][i]);
        return d != 0.0 && isfinite(d);
    }
}

// Block-Jacobi inverses read from assembled values (used when the node-centric gather
// does not apply): one thread per node.
template <int ND, int LAYOUT, typename T>
__global__ __launch_bounds__(256) void k_extract_binv(int64_t Nn, const int64_t *__restrict__ node_ptr,
                                                      const int32_t *__restrict__ bdiag,
                                                      const int64_t *__restrict__ row_ptr,
                                                      const int64_t *__restrict__ up_base,
                                                      const T *__restrict__ values, T *__restrict__ binv,
                                                      int *status) {
    const int64_t n = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (n >= Nn) return;
    double B[ND][ND];
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int c = 0; c < ND; ++c)
            B[i][c] = (LAYOUT == LAYOUT_SYM)
                          ? double(values[int64_t(ND) * ND * up_base[n] + i * ND + c])
                          : double(values[row_ptr[ND * n + i] + ND * (bdiag[n] - node_ptr[n]) + c]);
    if (!invert_block<ND>(B, binv + int64_t(ND) * ND * n)) atomicOr(status, ST_NAN);
}

// ------------------------------------------------------------------ tangent by rows
// The tangent of meshes whose nodes have at most 8 elements and 32 neighbours.  At a
// Gauss point every law here gives
//   K_e[(a,i),(b,k)] = sum_q sum_r C_ikr(a, q) dN_b,r(q),
//   C_ikr = P_i H_kr + R_i F_kr + Q_k H_ir + delta_ik (M dN_a)_r
// with dN the reference gradients, H, F, M matrices of the point (pulled back to the
// reference cube by J^{-T}) and P, Q, R vectors of node a, quadrature weight included:
//   neo-Hookean: H = F^{-T} J^{-T}, F = F J^{-T}, h = H dN_a, f = F dN_a,
//                P = aw h - c23 f, Q = bw h, R = -c23 h, M = cw J^{-1} J^{-T}
//   linear:      H = J^{-T}, P = lw h, Q = mw h, M = mw J^{-1} J^{-T}
//   Poisson:     M only.
// k_tangent_blocks: a wavefront takes 8 (FP32 values) or 4 (FP64 values) elements; a lane is
// one corner of an element's cube as in k_element_vec, evaluates its Gauss point once and
// leaves H, F c23, aw, bw (linear: H, lw, mw; Poisson: M) in LDS -- M dN_a is (3/2) (F c23)^T h, or
// H^T Q; then 16 lanes per element, two per node a (one for each half q2 of the points), sum C
// over the rule's factors -- dN_b,0 does not depend on q0, dN_b,1 not on q1, dN_b,2 not on q2 up
// to its sign, so 8 running sums per entry (i, k) hold what the 8 columns b need -- contract
// them with the one-dimensional shape values once and write the slot's row block, rows i
// one after the other.  Exchanges stay inside the wavefront: no block barrier.
// Arithmetic is FP64 for both types of values, and every entry is rounded once, when it is
// stored.  The sums of the factorised form are larger than the entries they leave; in FP32
// the blocks (a, b) and (b, a) round apart and the entries are further off than summed block by
// block.  |dK| / |K| and |K - K^T| / |K| of the FP32 tangent, factorised in FP32 / block by block
// in FP32 (k_element_tangent) / now: 40^3 neo-Hookean 1.28e-7, 5.1e-8 / 9.3e-8, 6.2e-8 / 4.0e-8, 0;
// 120x60x30 densities 9.7e-9, 1.4e-9 / 4.8e-9, 2.1e-9 / 2.1e-9, 0.
// What bounds it: at 100^3 with FP32 values (975 us) instruction issue -- 2,860 vector
// instructions per wavefront, two wavefronts per SIMD that issue 43% of the time each -- with the
// 2.4 GB it writes beside it; FP32 sums took 832 us.  (The 72 sums of all three rows at once
// spill: 2.1 ms.)  With FP64 values the 4.8 GB, 1,481 us.
// Whole tangent, element kernel and gather, with k_element_tangent -> now, us: 100^3 FP32
// 1,727 -> 1,773, FP64 3,776 -> 2,650 (linear 1,522 -> 1,507 and 3,570 -> 2,493, Poisson 492 -> 380
// and 1,291 -> 503); 37x29x23 64 -> 58 and 126 -> 69; 10^3 28.6 -> 21.5 and 38.6 -> 20.3.

// Numbers of a point in LDS: an odd count (one is unused for neo-Hookean and Poisson), with which
// the two elements and two halves that 32 lanes read at a time start in different banks (20
// for neo-Hookean: 64 us instead of 58 with FP32 values and 76 instead of 69 with FP64 at 37x29x23).
template <int MODEL>
constexpr int point_numbers() { return MODEL == FEM_POISSON ? 7 : (MODEL == FEM_LINEAR_ELASTIC ? 11 : 21); }
// Elements per wavefront: with FP64 values twice as many would leave two wavefronts per SIMD.
template <typename TV>
constexpr int wave_elems() { return sizeof(TV) == 4 ? 8 : 4; }

template <int MODEL, int ND, typename TV>
__global__ __launch_bounds__(kThreads, MODEL == FEM_NEO_HOOKEAN ? 2 : 3) void k_tangent_blocks(
    int64_t Ne, const double *__restrict__ coords, const int32_t *__restrict__ conn,
    const int32_t *__restrict__ kpos, Material mat, const double *__restrict__ theta, const double *__restrict__ u,
    TV *__restrict__ ke, int *status) {
    typedef double T;
    constexpr bool kNonlinear = MODEL == FEM_NEO_HOOKEAN;
    constexpr int BS = ND * ND, S = point_numbers<MODEL>(), W = 16 / int(sizeof(TV));
    constexpr int E = wave_elems<TV>();
    typedef TV vec __attribute__((ext_vector_type(16 / sizeof(TV))));
    // the points' numbers; and one row i of 32 slots on its way out
    constexpr int kRow = 8 * ND, kOut = ND == 1 ? 2 : 32 * kRow;
    __shared__ __align__(16) T lds[kThreads / 64][E * 8 * S];
    __shared__ __align__(16) TV out_lds[kThreads / 64][kOut];
    const int wave = threadIdx.x / 64, lane = threadIdx.x & 63;
    // Blocks of one XCD take adjacent elements: the slots of a node that share cache lines are
    // then completed in one L2 instead of leaving it as partial lines.
    const int64_t blk = int64_t(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const int64_t ew = (blk * (kThreads / 64) + wave) * E;  // first element of the wavefront
    if (ew >= Ne) return;  // wave-uniform; there are no block barriers
    int32_t my_slot;  // of this lane's node, -1 past the mesh
    // that of node a of element el (every lane takes part)
    auto slot = [&](int el, int a) -> int32_t {
        const int c = a ^ ((a >> 1) & 1);
        return __shfl(my_slot, el * 8 + (c ^ ((c & 4) ? 3 : 0)), 64);
    };
    {
        // lanes past the wavefront's or the mesh's elements repeat one and store nothing
        const int el = (lane >> 3) % E;
        const bool valid = lane < 8 * E && ew + el < Ne;
        ElemIds id;
        // corner of this lane, its node and its Gauss point as in k_element_vec
        const int l8 = lane & 7, c = l8 ^ ((l8 & 4) ? 3 : 0);
        id.a = c ^ ((c >> 1) & 1);
        id.el = el;
        id.valid = valid;
        id.e = ew + el < Ne ? ew + el : Ne - 1;
        const int64_t e = id.e;
        T X[3], U[ND];
        load_node<ND, kNonlinear ? LOAD_FIELD | LOAD_REL : LOAD_COORDS>(coords, conn, u, nullptr, id, X, U);
        const T mod = modulus(mat, theta[e]);
        // (the slots too, before the first store: a load after one would wait for it)
        my_slot = kpos[e * 8 + id.a];
        if (!valid) my_slot = -1;
        // J and the gradients without the factor p^2 / 2 of every column and the sign s_k of column k
        T J[3][3], Gr[3][3] = {};
#pragma unroll
        for (int i = 0; i < 3; ++i) corner_grad(X[i], J[i]);
        if constexpr (kNonlinear)
#pragma unroll
            for (int i = 0; i < ND; ++i) corner_grad(U[i], Gr[i]);
        const T dj = det3(J);
        const T d = (__popc(c) & 1) ? kCornerDet * dj : -kCornerDet * dj;
        bool mat_ok = true;
        T B[3][3];  // J^{-T}, likewise
        inv_transpose3(J, dj, B);
        // Weight of the point: the factors common to all columns b (every 1-D shape value below is
        // taken relative to the larger one) and the (2 / p^2)^2 left out of the two B of each term.
        const T wq = T(kPointWeight) * d;
        T out[S] = {};
        auto put_matrix = [&](int at, const T A[3][3]) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int r = 0; r < 3; ++r) out[at + 3 * i + r] = A[i][r];
        };
        auto times_b = [&](const T A[3][3], T R[3][3]) {  // A J^{-T}
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int r = 0; r < 3; ++r) R[i][r] = A[i][0] * B[0][r] + A[i][1] * B[1][r] + A[i][2] * B[2][r];
        };
        T G[3][3];
        if constexpr (kNonlinear)
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) G[i][j] = Gr[i][0] * B[j][0] + Gr[i][1] * B[j][1] + Gr[i][2] * B[j][2];
        // The signs s_0 and s_1 of the columns.  The third column stays without: its axis is reversed
        // where q2 = 0, so that columns b2 = 0 enter with the same sign as b2 = 1.
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            B[i][0] = (c & 1) ? B[i][0] : -B[i][0];
            B[i][1] = (c & 2) ? B[i][1] : -B[i][1];
        }
        if constexpr (MODEL == FEM_NEO_HOOKEAN) {
            NHState<T> st;
            mat_ok = nh_state(G, mod, T(mat.bulk_ratio), st);
            T R[3][3];
            times_b(st.H, R);
            put_matrix(0, R);
            const T cw = wq * st.c, c23 = T(2.0 / 3.0) * cw;
            times_b(st.F, R);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int r = 0; r < 3; ++r) R[i][r] *= c23;
            put_matrix(9, R);
            out[18] = wq * st.alpha;
            out[19] = wq * st.beta;
        } else if constexpr (MODEL == FEM_LINEAR_ELASTIC) {
            const T nu = T(mat.nu);
            const T lw = wq * mod * nu / ((T(1) + nu) * (T(1) - T(2) * nu)), mw = wq * mod / (T(2) * (T(1) + nu));
            put_matrix(0, B);
            out[9] = lw;
            out[10] = mw;
        } else {
            constexpr int pr[6][2] = {{0, 0}, {1, 1}, {2, 2}, {1, 2}, {0, 2}, {0, 1}};
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const int r = pr[q][0], t = pr[q][1];
                out[q] = wq * mod * (B[0][r] * B[0][t] + B[1][r] * B[1][t] + B[2][r] * B[2][t]);
            }
        }
        if (valid && (!(d > T(0)) || !mat_ok))
            atomicOr(status, (!(d > T(0)) ? ST_MESH : 0) | (!mat_ok ? ST_INVERTED : 0));
        if (lane < 8 * E) {
            T *dst = lds[wave] + (el * 8 + c) * S;
#pragma unroll
            for (int q = 0; q < S; ++q) dst[q] = out[q];
        }
        wave_lds_handoff();
    }
    const int half = lane & 1, a = (lane >> 1) & 7;
    const T lp = T(0.78867513459481288225), lm = T(0.21132486540518711775);  // (1 +- 1/sqrt(3)) / 2
    const bool ax = (a ^ (a >> 1)) & 1, ay = (a >> 1) & 1, az = (a >> 2) & 1;
    // the sign of dN_a,2 goes with the reversed axis
    const T hx = ax ? T(0.5) : T(-0.5), hy = ay ? T(0.5) : T(-0.5), hz = (az == bool(half)) ? T(0.5) : T(-0.5);
    const T l2 = (az == bool(half)) ? lp : lm, t = lm / lp;
#pragma unroll 1
    for (int round = 0; round < E / 4; ++round) {
        const int el = 4 * round + (lane >> 4);
        int at = (el * 8 + 4 * half) * S;
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            // (an opaque offset: the numbers are read from LDS again for every row
            // instead of being carried along in registers)
            asm volatile("" : "+v"(at));
            const T *pt = lds[wave] + at;
            T S0[2][ND], S1[2][ND], S2[2][2][ND];
#pragma unroll
            for (int q1 = 0; q1 < 2; ++q1)
#pragma unroll
                for (int q0 = 0; q0 < 2; ++q0) {
                    const T *st = pt + (2 * q1 + q0) * S;
                    const T l0 = (ax == bool(q0)) ? lp : lm, l1 = (ay == bool(q1)) ? lp : lm;
                    const T dN[3] = {hx * l1 * l2, hy * l0 * l2, hz * l0 * l1};
                    // the running sums of the three directions; first: they start at this point
                    auto first = [&](int r) { return r == 2 || (r == 0 ? q0 : q1) == 0; };
                    auto sum = [&](int k, int r) -> T { return r == 0 ? S0[q1][k] : S1[q0][k]; };
                    auto put = [&](int k, int r, T v) {
                        if (r == 0) S0[q1][k] = v;
                        else if (r == 1) S1[q0][k] = v;
                        else S2[q0][q1][k] = v;
                    };
                    if constexpr (MODEL == FEM_POISSON) {
                        const T gb[3] = {st[0] * dN[0] + st[5] * dN[1] + st[4] * dN[2],
                                         st[5] * dN[0] + st[1] * dN[1] + st[3] * dN[2],
                                         st[4] * dN[0] + st[3] * dN[1] + st[2] * dN[2]};
#pragma unroll
                        for (int r = 0; r < 3; ++r) put(0, r, first(r) ? gb[r] : sum(0, r) + gb[r]);
                    } else {
                        constexpr bool kF = MODEL != FEM_LINEAR_ELASTIC;
                        const T *H = st, *F = st + 9;
                        T h[3], Q[3];
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            h[k] = H[3 * k] * dN[0] + H[3 * k + 1] * dN[1] + H[3 * k + 2] * dN[2];
                            Q[k] = st[kF ? 19 : 10] * h[k];
                        }
                        T gb[3];  // M dN_a
#pragma unroll
                        for (int r = 0; r < 3; ++r)
                            gb[r] = kF ? T(1.5) * (F[r] * h[0] + F[3 + r] * h[1] + F[6 + r] * h[2])
                                       : H[r] * Q[0] + H[3 + r] * Q[1] + H[6 + r] * Q[2];
                        const T *Hi = H + 3 * i, *Fi = F + 3 * i;
                        const T fi = kF ? Fi[0] * dN[0] + Fi[1] * dN[1] + Fi[2] * dN[2] : T(0);
                        T P, R = T(0);
                        if constexpr (MODEL == FEM_NEO_HOOKEAN) {
                            P = st[18] * h[i] - fi;
                            R = -h[i];
                        } else {
                            P = st[9] * h[i];
                        }
#pragma unroll
                        for (int k = 0; k < 3; ++k)
#pragma unroll
                            for (int r = 0; r < 3; ++r) {
                                T v;
                                if (first(r)) v = k == i ? fma(P, H[3 * k + r], gb[r]) : P * H[3 * k + r];
                                else v = fma(P, H[3 * k + r], k == i ? sum(k, r) + gb[r] : sum(k, r));
                                if constexpr (kF) v = fma(R, F[3 * k + r], v);
                                put(k, r, fma(Q[k], Hi[r], v));
                            }
                    }
                }
            // Columns b = (b0, b1, b2): dN_b,0 = s0 l_b1 l_b2 / 2 and so on; with every l over lp (1 or
            // t) and lp^2 / 2 in the weights, half h adds l_b2(h) A + B to column b, where
            //   A[b0][b1] = s0 sum_q1 l_b1 S0 + s1 sum_q0 l_b0 S1,  B[b0][b1] = sum l_b0 l_b1 S2
            // for b2 = h, and l_b2(h) A - B for the other.  Lane h keeps b2 = h and hands its part
            // of the other to its neighbour.  Nodes in HEX8 order: (b0, b1) = 00, 10, 11, 01.
            T o[4 * ND];
#pragma unroll
            for (int k = 0; k < ND; ++k) {
                const T u0 = fma(t, S0[1][k], S0[0][k]), u1 = fma(t, S0[0][k], S0[1][k]);
                const T w0 = fma(t, S1[1][k], S1[0][k]), w1 = fma(t, S1[0][k], S1[1][k]);
                const T v00 = fma(t, S2[1][0][k], S2[0][0][k]), v10 = fma(t, S2[0][0][k], S2[1][0][k]);
                const T v01 = fma(t, S2[1][1][k], S2[0][1][k]), v11 = fma(t, S2[0][1][k], S2[1][1][k]);
                const T A[4] = {-u0 - w0, u0 - w1, u1 + w1, w0 - u1};
                const T B[4] = {fma(t, v01, v00), fma(t, v11, v10), fma(t, v10, v11), fma(t, v00, v01)};
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    o[b * ND + k] = (A[b] + B[b]) + dpp_read<kDppXor1>(fma(t, A[b], -B[b]));
            }
            // Row i of a slot is 8 * ND consecutive values.  The wavefront's 32 rows go through
            // LDS so that neighbouring lanes store neighbouring 16-byte pieces (stored straight
            // from each lane's registers they took as long again as the whole kernel).
            if constexpr (ND == 1) {
                const int32_t k = slot(el, a);
                if (k >= 0) {
                    TV *row = ke + int64_t(k) * 8 * BS + half * 4;
#pragma unroll
                    for (int v = 0; v < 4; ++v) row[v] = TV(o[v]);
                }
            } else {
                TV *stage = out_lds[wave];
#pragma unroll
                for (int v = 0; v < 4 * ND / W; ++v) {
                    vec x;
#pragma unroll
                    for (int w = 0; w < W; ++w) x[w] = TV(o[v * W + w]);
                    reinterpret_cast<vec *>(stage + lane * 4 * ND)[v] = x;
                }
                wave_lds_handoff();
                constexpr int kP = kRow / W;  // pieces per row
#pragma unroll
                for (int t = 0; t < 32 * kP / 64; ++t) {
                    const int p = lane + 64 * t, sl = p / kP;
                    const int32_t k = slot(4 * round + sl / 8, sl % 8);
                    const vec x = reinterpret_cast<const vec *>(stage)[p];
                    if (k >= 0)
                        reinterpret_cast<vec *>(ke + int64_t(k) * 8 * BS + i * kRow)[p - sl * kP] = x;
                }
                wave_lds_handoff();  // before the next row is staged
            }
        }
    }
}

constexpr int kGatherMaxDeg = 32;  // neighbours of a node on the row path
constexpr int kGatherMaxInc = 8;   // and its elements

// The rows of two consecutive nodes per wavefront, 32 lanes each.  The slots of a node
// (and of the next one) are one contiguous run of the element kernel's output (BLOCKS: of
// k_element_tangent's, block after block; else k_tangent_blocks', row after row): the wavefront
// copies it to LDS, lane j of a half sums what belongs to neighbour block j -- a 64-bit
// mask per block (bit 8 * slot + b), built from the slots' target bytes, lists its
// contributions in element order -- applies the symmetric Dirichlet elimination and
// writes each CSR value once, with the node's Jacobi diagonal or block inverse.  No
// read-modify-write of an image and no block barrier.
// What bounds it: at 100^3 in FP32 its 2.3 GB in and 1.0 GB out, 5.1 TB/s (650 us; slot by
// slot additions into an LDS image of the rows took 1,079 us); FP64, 37x29x23: 39 -> 28 us.
template <int ND, int LAYOUT, bool BLOCKS, typename T>
__global__ __launch_bounds__(kThreads) void k_gather_rows(int64_t Nn, const int64_t *__restrict__ node_ptr,
                                                          const uint8_t *__restrict__ nb_bits,
                                                          const int64_t *__restrict__ ne_ptr,
                                                          const uint8_t *__restrict__ tgt,
                                                          const int32_t *__restrict__ bdiag,
                                                          const int64_t *__restrict__ up_base,
                                                          const uint8_t *__restrict__ mask, const T *__restrict__ ke,
                                                          T *__restrict__ values, T *__restrict__ dinv, int bj,
                                                          int *status) {
    constexpr int BS = ND * ND, W = 16 / int(sizeof(T)), kSlot = 8 * BS;
    constexpr int kMaxT = 2 * kGatherMaxInc * kSlot;            // values of a pair of nodes
    constexpr int kPieces = (kMaxT / W + 63) / 64;              // 16-byte pieces per lane
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    __shared__ __align__(16) T run[kThreads / 64][kMaxT];
    __shared__ unsigned long long mset[kThreads / 32][kGatherMaxDeg];
    const int wave = threadIdx.x / 64, lane64 = threadIdx.x & 63, lane = threadIdx.x & 31, grp = threadIdx.x >> 5;
    const int64_t n0 = (int64_t(blockIdx.x) * (kThreads / 64) + wave) * 2;
    if (n0 >= Nn) return;  // wave-uniform; there are no block barriers
    const int64_t k0 = ne_ptr[n0], kmid = ne_ptr[n0 + 1], k1 = n0 + 1 < Nn ? ne_ptr[n0 + 2] : kmid;
    const int pieces = int(k1 - k0) * kSlot / W;
    const vec *src = reinterpret_cast<const vec *>(ke + k0 * kSlot);
    vec buf[kPieces];
#pragma unroll
    for (int t = 0; t < kPieces; ++t) {
        const int i = lane64 + 64 * t;
        buf[t] = src[i < pieces ? i : 0];
    }
    // this half's node; the second half of an odd last pair idles on the first one
    const bool live = n0 + (grp & 1) < Nn;
    const int64_t n = live ? n0 + (grp & 1) : n0;
    const int64_t kn = live && (grp & 1) ? kmid : k0;
    const int pairs = 8 * int((live && (grp & 1) ? k1 : kmid) - kn);
    const int64_t nb0 = node_ptr[n];
    const int deg = int(node_ptr[n + 1] - nb0), jd = int(bdiag[n] - nb0);
    const bool act = lane < deg;
    const int colbits = nb_bits[nb0 + (act ? lane : 0)];
    int rowbits = 0;
    if (mask)
#pragma unroll
        for (int c = 0; c < ND; ++c) rowbits |= int(mask[ND * n + c] != 0) << c;
    const int t0 = tgt[kn * 8 + (lane < pairs ? lane : 0)], t1 = tgt[kn * 8 + (lane + 32 < pairs ? lane + 32 : 0)];
    mset[grp][lane] = 0;
    wave_lds_handoff();
    if (lane < pairs) atomicOr(&mset[grp][t0], 1ull << lane);
    if (lane + 32 < pairs) atomicOr(&mset[grp][t1], 1ull << (lane + 32));
#pragma unroll
    for (int t = 0; t < kPieces; ++t)
        if (lane64 + 64 * t < pieces) reinterpret_cast<vec *>(run[wave])[lane64 + 64 * t] = buf[t];
    wave_lds_handoff();
    unsigned long long m = act ? mset[grp][lane] : 0;
    // the diagonal block has twice as many contributions as any other of a structured
    // mesh: a free lane takes those of its last four slots
    const bool split = deg < 32;
    if (split) {
        if (lane == jd) m &= 0xffffffffull;
        else if (lane == 31) m = mset[grp][jd] & ~0xffffffffull;
    }
    T acc[BS];
#pragma unroll
    for (int c = 0; c < BS; ++c) acc[c] = T(0);
    const T *mine = run[wave] + (kn - k0) * kSlot;
    while (m) {  // ascending slots: element order
        const int l = __builtin_ctzll(m);
        m &= m - 1;
        const T *o = mine + (l >> 3) * kSlot + (l & 7) * (BLOCKS ? BS : ND);
#pragma unroll
        for (int i = 0; i < ND; ++i)
#pragma unroll
            for (int c = 0; c < ND; ++c) acc[i * ND + c] += o[i * (BLOCKS ? ND : 8 * ND) + c];
    }
    if (split)
#pragma unroll
        for (int c = 0; c < BS; ++c) {
            const T up = __shfl(acc[c], 31, 32);
            if (lane == jd) acc[c] += up;
        }
    if (!act || !live) return;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int c = 0; c < ND; ++c) {
            if (((rowbits >> i) | (colbits >> c)) & 1) acc[i * ND + c] = (lane == jd && i == c) ? T(1) : T(0);
            bad |= !isfinite(acc[i * ND + c]);
        }
#pragma unroll
    for (int i = 0; i < ND; ++i) {
        T *dst = (LAYOUT == LAYOUT_SYM) ? values + int64_t(BS) * (up_base[n] + lane - jd) + i * ND
                                        : values + int64_t(BS) * nb0 + int64_t(i) * ND * deg + ND * lane;
        if (LAYOUT != LAYOUT_SYM || lane >= jd)
#pragma unroll
            for (int c = 0; c < ND; ++c) dst[c] = acc[i * ND + c];
    }
    if (dinv && lane == jd) {
        if (!bj) {
#pragma unroll
            for (int c = 0; c < ND; ++c) {
                bad |= !(acc[c * ND + c] != T(0));
                dinv[ND * n + c] = T(1) / acc[c * ND + c];
            }
        } else {
            double B[ND][ND];
#pragma unroll
            for (int i = 0; i < ND; ++i)
#pragma unroll
                for (int c = 0; c < ND; ++c) B[i][c] = double(acc[i * ND + c]);
            bad |= !invert_block<ND>(B, dinv + int64_t(BS) * n);
        }
    }
    if (bad) atomicOr(status, ST_NAN);
}

template <int ND, int LAYOUT, typename T>
__global__ __launch_bounds__(256) void k_extract_dinv(int64_t N, const int64_t *__restrict__ node_ptr,
                                                      const int32_t *__restrict__ bdiag,
                                                      const int64_t *__restrict__ row_ptr,
                                                      const int64_t *__restrict__ up_base,
                                                      const T *__restrict__ values, T *__restrict__ dinv,
                                                      int *status) {
    int64_t d = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (d >= N) return;
    int64_t n = d / ND;
    int i = int(d - n * ND);
    T v = (LAYOUT == LAYOUT_SYM) ? values[ND * ND * up_base[n] + (ND + 1) * i]
                                 : values[row_ptr[d] + ND * (bdiag[n] - node_ptr[n]) + i];
    if (!(v != T(0)) || !isfinite(v)) atomicOr(status, ST_NAN);
    dinv[d] = T(1) / v;
}

inline unsigned grid_for(int64_t n, int threads) { return unsigned((n + threads - 1) / threads); }

}  // namespace

// ------------------------------------------------------------------ launchers
#define FEM_DISPATCH_MODEL(h, CALL)                                                                  \
    switch ((h)->mat.model) {                                                                        \
    case FEM_POISSON: { constexpr int MODEL = FEM_POISSON; constexpr int ND = 1; CALL; break; }      \
    case FEM_LINEAR_ELASTIC: { constexpr int MODEL = FEM_LINEAR_ELASTIC; constexpr int ND = 3; CALL; break; } \
    case FEM_J2_PLASTIC: { constexpr int MODEL = FEM_J2_PLASTIC; constexpr int ND = 3; CALL; break; }        \
    default: { constexpr int MODEL = FEM_NEO_HOOKEAN; constexpr int ND = 3; CALL; break; }          \
    }

void launch_residual(const fem_handle *h, const double *u, const double *theta, double lf, double *scratch,
                     double *r, hipStream_t s) {
    const Graph &g = h->g;
    if (g.Ne == 0) {
        FEM_HIP(hipMemsetAsync(r, 0, g.N * sizeof(double), s));
        return;
    }
    unsigned gridE = grid_for(g.Ne, kElemsPerBlock);
    FEM_DISPATCH_MODEL(h, {
        hipLaunchKernelGGL((k_element_vec<MODEL, ND, VEC_RESIDUAL>), dim3(gridE), dim3(kThreads), 0, s, g.Ne,
                           h->m.coords, h->m.conn, g.kpos, h->m.mask, h->mat, theta, u, nullptr, h->hist, scratch,
                           h->status);
        hipLaunchKernelGGL((k_gather_vec<ND, VEC_RESIDUAL>), dim3(grid_for(g.Nn, 32)), dim3(256), 0, s, g.Nn,
                           g.ne_ptr, scratch, h->m.mask, h->m.fext, lf, nullptr, r, h->status);
    });
    FEM_HIP(hipGetLastError());
}

void launch_apply_tangent(const fem_handle *h, const double *u, const double *theta, const double *v,
                          double *scratch, double *y, hipStream_t s) {
    const Graph &g = h->g;
    if (g.Ne == 0) {
        FEM_HIP(hipMemcpyAsync(y, v, g.N * sizeof(double), hipMemcpyDeviceToDevice, s));
        return;
    }
    unsigned gridE = grid_for(g.Ne, kElemsPerBlock);
    FEM_DISPATCH_MODEL(h, {
        hipLaunchKernelGGL((k_element_vec<MODEL, ND, VEC_JVP>), dim3(gridE), dim3(kThreads), 0, s, g.Ne, h->m.coords,
                           h->m.conn, g.kpos, h->m.mask, h->mat, theta, u, v, h->hist, scratch, h->status);
        hipLaunchKernelGGL((k_gather_vec<ND, VEC_JVP>), dim3(grid_for(g.Nn, 32)), dim3(256), 0, s, g.Nn, g.ne_ptr,
                           scratch, h->m.mask, nullptr, 0.0, v, y, h->status);
    });
    FEM_HIP(hipGetLastError());
}

void launch_lift(const fem_handle *h, const double *u, const double *theta, const double *v, double *scratch,
                 double *y, hipStream_t s) {
    const Graph &g = h->g;
    if (g.Ne == 0) return;
    unsigned gridE = grid_for(g.Ne, kElemsPerBlock);
    FEM_DISPATCH_MODEL(h, {
        hipLaunchKernelGGL((k_element_vec<MODEL, ND, VEC_LIFT>), dim3(gridE), dim3(kThreads), 0, s, g.Ne,
                           h->m.coords, h->m.conn, g.kpos, h->m.mask, h->mat, theta, u, v, h->hist, scratch, h->status);
        hipLaunchKernelGGL((k_gather_vec<ND, VEC_LIFT>), dim3(grid_for(g.Nn, 32)), dim3(256), 0, s, g.Nn, g.ne_ptr,
                           scratch, h->m.mask, nullptr, 0.0, v, y, h->status);
    });
    FEM_HIP(hipGetLastError());
}

void launch_mass(const fem_handle *h, const double *x, double *scratch, double *y, hipStream_t s) {
    const Graph &g = h->g;
    if (g.Ne == 0) {
        FEM_HIP(hipMemsetAsync(y, 0, g.N * sizeof(double), s));
        return;
    }
    unsigned gridE = grid_for(g.Ne, kElemsPerBlock);
    if (g.nd == 1) {
        hipLaunchKernelGGL((k_element_mass<1>), dim3(gridE), dim3(kThreads), 0, s, g.Ne, h->m.coords, h->m.conn,
                           g.kpos, x, scratch, h->status);
        hipLaunchKernelGGL((k_gather_vec<1, VEC_MASS>), dim3(grid_for(g.Nn, 32)), dim3(256), 0, s, g.Nn, g.ne_ptr,
                           scratch, nullptr, nullptr, 0.0, nullptr, y, h->status);
    } else {
        hipLaunchKernelGGL((k_element_mass<3>), dim3(gridE), dim3(kThreads), 0, s, g.Ne, h->m.coords, h->m.conn,
                           g.kpos, x, scratch, h->status);
        hipLaunchKernelGGL((k_gather_vec<3, VEC_MASS>), dim3(grid_for(g.Nn, 32)), dim3(256), 0, s, g.Nn, g.ne_ptr,
                           scratch, nullptr, nullptr, 0.0, nullptr, y, h->status);
    }
    FEM_HIP(hipGetLastError());
}

void launch_j2_commit(const fem_handle *h, const double *u, const double *theta, hipStream_t s) {
    const Graph &g = h->g;
    if (g.Ne == 0 || h->mat.model != FEM_J2_PLASTIC) return;
    hipLaunchKernelGGL(k_j2_commit, dim3(grid_for(g.Ne, kElemsPerBlock)), dim3(kThreads), 0, s, g.Ne, h->m.coords,
                       h->m.conn, h->mat, theta, u, h->hist);
    FEM_HIP(hipGetLastError());
}

size_t j2_partials_count(int64_t n_elems) { return size_t(grid_for(n_elems, kElemsPerBlock)) * 7; }

void j2_average_stress(fem_handle *h, double out[6], hipStream_t s) {
    const Graph &g = h->g;
    for (int c = 0; c < 6; ++c) out[c] = 0.0;
    if (g.Ne == 0) return;
    const unsigned grid = grid_for(g.Ne, kElemsPerBlock);
    hipLaunchKernelGGL(k_j2_average, dim3(grid), dim3(kThreads), 0, s, g.Ne, h->m.coords, h->m.conn, h->hist,
                       h->hist_partials);
    FEM_HIP(hipGetLastError());
    std::vector<double> hp(size_t(grid) * 7);
    FEM_HIP(hipMemcpyAsync(hp.data(), h->hist_partials, hp.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    FEM_HIP(hipStreamSynchronize(s));
    double t[7] = {0, 0, 0, 0, 0, 0, 0};
    for (unsigned b = 0; b < grid; ++b)
        for (int c = 0; c < 7; ++c) t[c] += hp[size_t(b) * 7 + c];
    for (int c = 0; c < 6; ++c) out[c] = t[c] / t[6];
}

void launch_vjp(const fem_handle *h, const double *u, const double *theta, const double *lam, double *gout,
                hipStream_t s) {
    const Graph &g = h->g;
    if (g.Ne == 0) return;
    if (h->mat.model == FEM_J2_PLASTIC) throw Error(FEM_EINVAL, "the parameter VJP is not defined for FEM_J2_PLASTIC");
    unsigned gridE = grid_for(g.Ne, kElemsPerBlock);
    FEM_DISPATCH_MODEL(h, {
        hipLaunchKernelGGL((k_element_vec<MODEL, ND, VEC_VJP>), dim3(gridE), dim3(kThreads), 0, s, g.Ne, h->m.coords,
                           h->m.conn, g.kpos, h->m.mask, h->mat, theta, u, lam, nullptr, gout, h->status);
    });
    FEM_HIP(hipGetLastError());
}

// The element blocks of the row gather.  J2 keeps the form that evaluates the return map at
// the strains of its residual, rounding included: with the factorised gradients a point that
// the history put on the yield surface could be elastic in one and plastic in the other, and
// past the limit load CG then met matrices it could not solve (48x48x96 cylinder, loading and
// unloading in 20 steps: 20,000 iterations without convergence; with this form 5.5 s).
template <int MODEL, int ND, typename T>
static void launch_element_blocks(const fem_handle *h, const double *u, const double *theta, T *ke, hipStream_t s) {
    const Graph &g = h->g;
    if constexpr (MODEL == FEM_J2_PLASTIC)
        hipLaunchKernelGGL((k_element_tangent<MODEL, ND, T>), dim3(grid_for(g.Ne, kElemsPerBlock)), dim3(kThreads), 0, s,
                           g.Ne, h->m.coords, h->m.conn, g.kpos, h->mat, theta, u, h->hist, ke, h->status);
    else
        hipLaunchKernelGGL((k_tangent_blocks<MODEL, ND, T>),
                           dim3((grid_for(g.Ne, wave_elems<T>() * kThreads / 64) + 7) / 8 * 8), dim3(kThreads), 0, s,
                           g.Ne, h->m.coords, h->m.conn, g.kpos, h->mat, theta, u, ke, h->status);
}

template <typename T>
void launch_tangent(const fem_handle *h, const double *u, const double *theta, T *ke, T *values, T *dinv,
                    hipStream_t s, int layout, int precond) {
    const int bj = precond == FEM_PRECOND_BLOCK_JACOBI;
    const Graph &g = h->g;
    if (g.Ne == 0) return;
    // Nodes beyond 8 elements or 32 neighbours (fans, irregular block corners) do not fit
    // the row gather's masks and lanes: element matrices and the per-block gather.
    const bool by_rows = g.tgt != nullptr && g.max_deg <= kGatherMaxDeg && g.max_inc <= kGatherMaxInc;
    FEM_DISPATCH_MODEL(h, {
        if (by_rows) {
            (launch_element_blocks<MODEL, ND, T>(h, u, theta, ke, s));
            const dim3 grid(grid_for(g.Nn, 2 * kThreads / 64));
            if (layout == LAYOUT_SYM)
                hipLaunchKernelGGL((k_gather_rows<ND, LAYOUT_SYM, MODEL == FEM_J2_PLASTIC, T>), grid, dim3(kThreads), 0, s, g.Nn, g.node_ptr,
                                   g.nb_bits, g.ne_ptr, g.tgt, g.bdiag, g.up_base, h->m.mask, ke, values, dinv, bj,
                                   h->status);
            else
                hipLaunchKernelGGL((k_gather_rows<ND, LAYOUT_CSR, MODEL == FEM_J2_PLASTIC, T>), grid, dim3(kThreads), 0, s, g.Nn, g.node_ptr,
                                   g.nb_bits, g.ne_ptr, g.tgt, g.bdiag, g.up_base, h->m.mask, ke, values, dinv, bj,
                                   h->status);
        } else {
            hipLaunchKernelGGL((k_element_tangent<MODEL, ND, T>), dim3(grid_for(g.Ne, kElemsPerBlock)), dim3(kThreads),
                               0, s, g.Ne, h->m.coords, h->m.conn, g.kpos, h->mat, theta, u, h->hist, ke, h->status);
            if (layout == LAYOUT_SYM)
                hipLaunchKernelGGL((k_gather_values<ND, LAYOUT_SYM, T>), dim3(grid_for(g.nnzb * ND, 256)), dim3(256),
                                   0, s, g.nnzb, g.node_ptr, g.node_nb, g.blk_row, g.blk_ptr, g.blk_src, g.row_ptr,
                                   g.bdiag, g.up_base, h->m.mask, ke, values, h->status);
            else
                hipLaunchKernelGGL((k_gather_values<ND, LAYOUT_CSR, T>), dim3(grid_for(g.nnzb * ND, 256)), dim3(256),
                                   0, s, g.nnzb, g.node_ptr, g.node_nb, g.blk_row, g.blk_ptr, g.blk_src, g.row_ptr,
                                   g.bdiag, g.up_base, h->m.mask, ke, values, h->status);
        }
    });
    FEM_HIP(hipGetLastError());
    if (dinv && !by_rows) {
        if (!bj) {
            launch_extract_dinv<T>(h, values, dinv, s, layout);
        } else {
#define FEM_BINV(ND, LY)                                                                                           \
    hipLaunchKernelGGL((k_extract_binv<ND, LY, T>), dim3(grid_for(g.Nn, 256)), dim3(256), 0, s, g.Nn, g.node_ptr, \
                       g.bdiag, g.row_ptr, g.up_base, values, dinv, h->status)
            if (g.nd == 1) {
                if (layout == LAYOUT_SYM) FEM_BINV(1, LAYOUT_SYM);
                else FEM_BINV(1, LAYOUT_CSR);
            } else {
                if (layout == LAYOUT_SYM) FEM_BINV(3, LAYOUT_SYM);
                else FEM_BINV(3, LAYOUT_CSR);
            }
#undef FEM_BINV
            FEM_HIP(hipGetLastError());
        }
    }
}

template <typename T>
void launch_extract_dinv(const fem_handle *h, const T *values, T *dinv, hipStream_t s, int layout) {
    const Graph &g = h->g;
    if (g.N == 0) return;
#define FEM_DINV(ND, LY)                                                                                         \
    hipLaunchKernelGGL((k_extract_dinv<ND, LY, T>), dim3(grid_for(g.N, 256)), dim3(256), 0, s, g.N, g.node_ptr,  \
                       g.bdiag, g.row_ptr, g.up_base, values, dinv, h->status)
    if (g.nd == 1) {
        if (layout == LAYOUT_SYM) FEM_DINV(1, LAYOUT_SYM);
        else FEM_DINV(1, LAYOUT_CSR);
    } else {
        if (layout == LAYOUT_SYM) FEM_DINV(3, LAYOUT_SYM);
        else FEM_DINV(3, LAYOUT_CSR);
    }
#undef FEM_DINV
    FEM_HIP(hipGetLastError());
}

template void launch_tangent<float>(const fem_handle *, const double *, const double *, float *, float *, float *,
                                    hipStream_t, int, int);
template void launch_tangent<double>(const fem_handle *, const double *, const double *, double *, double *,
                                     double *, hipStream_t, int, int);
template void launch_extract_dinv<float>(const fem_handle *, const float *, float *, hipStream_t, int);
template void launch_extract_dinv<double>(const fem_handle *, const double *, double *, hipStream_t, int);

}  // namespace fem
