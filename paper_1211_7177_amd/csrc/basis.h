// Basis evaluation shared by the forward and adjoint expansion kernels:
// normalised associated Legendre recurrences and the regular solid harmonics
// R_n^m(d) = j_n(k|d|) Y_n^m(d/|d|) (eqs. 2.14-2.15), with constants tabulated
// on the host at plan time.
#pragma once
#include "common.h"

namespace fmb {

// ---------------------------------------------------------------- basis
// Recurrence constants of the normalised associated Legendre functions and of
// the gradient of R_n^m, tabulated on the host at plan time (BasisTab layout
// below) so that the per-node loops carry no square roots or divisions.
//   Q_m^m = qmm[m],
//   Q_n^m = la[n][m] (x Q_{n-1}^m - lb[n][m] Q_{n-2}^m)            (n > m, Q_{m-1}^m = 0)
template <typename T>
struct BasisTab {
    const T *la, *lb, *qmm;          // [(N+1)^2] (row n, column m), [(N+1)^2], [N+1]
    const T *gco;                    // [P2][6] gradient coefficients of coefficient idx (mu = -m)
    int N;
};

template <typename T>
__device__ inline BasisTab<T> basis_tab(const T *tab, int N) {
    BasisTab<T> b;
    const int NN = (N + 1) * (N + 1);
    b.la = tab;
    b.lb = tab + NN;
    b.qmm = tab + 2 * NN;
    b.gco = tab + 2 * NN + (N + 1);
    b.N = N;
    return b;
}

// The kernels at the leaves (sources to multipoles, local expansions to nodes)
// are products with the real matrix
//   E[(n, m, cos | sin)][node] = (-1)^m Q_n^m(cos th) Re | Im (sin th e^{i ph})^m,
//   R_n^{+-m} = j_n(k r) (E_cos +- i E_sin),
// on the matrix cores.  A lane of a 16x16x4 step owns one (order, cos | sin) and
// one node and runs the recurrence of Q_n^m over n in registers, so the basis is
// never stored.
template <typename T>
struct Mma16;
// lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; register q of lane l
// holds D[row(l / 16, q)][l % 16]; kq_of and q_of invert row
template <>
struct Mma16<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(double a, double b, v4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row(int kq, int q) { return 4 * q + kq; }
    __device__ static int kq_of(int r) { return r & 3; }
    __device__ static int q_of(int r) { return r >> 2; }
};
template <>
struct Mma16<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(float a, float b, v4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int row(int kq, int q) { return 4 * kq + q; }
    __device__ static int kq_of(int r) { return r >> 2; }
    __device__ static int q_of(int r) { return r & 3; }
};

// x of the neighbouring lane (re <-> im)
__device__ __forceinline__ float lane_swap(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_swap(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0xB1, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0xB1, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Barrier that orders LDS accesses only: global loads and stores in flight stay in flight.
__device__ __forceinline__ void leaf_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS that a block of the leaf kernels may have (a CU's, less 1 KB); launches that take
// more than the default 64 KB ask for all of it, so that plans of other orders set the same value
constexpr size_t LEAF_LDS_MAX = 160 * 1024 - 1024;
template <typename K>
inline void leaf_lds_limit(K kern, size_t bytes) {
    FMB_REQUIRE(bytes <= LEAF_LDS_MAX, "a leaf kernel's tables exceed a block's LDS");
    if (bytes > 65536)
        FMB_CHECK_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                          (int)LEAF_LDS_MAX));
}

// What the kernels at the leaves need of a node, laid out at plan time: the direction
// from its leaf's centre (cos th, sin th e^{i ph}), z = k r and the heads g_p, g_{p+1}
// of the recurrence below.  The library sine, the divisions and the start above degree
// p stay out of the kernels, where few lanes ran them and the rest of the block waited
// (10 reals a node: 40 or 80 B against the 56 or 112 B of its source record).
template <typename T>
struct LeafNode {
    T x, pad;
    cx<T> w, z, g0, g1;
};

// 1 / (2 n + 1) and 1 / ((2 n + 1)(2 n + 3)), n <= N
template <typename T>
__device__ inline void leaf_inv_table(int N, cx<T> *inv) {
    for (int i = threadIdx.x; i <= N; i += blockDim.x) inv[i] = mk(T(1) / (2 * i + 1), T(1) / ((2 * i + 1) * (2 * i + 3)));
}

// j_n(z), n <= N <= p, of one node into out[n * stride].  j_n = z^n / (2n+1)!! g_n with
// g_{n-1} = g_n - z^2 / ((2n+1)(2n+3)) g_{n+1}: g stays near one, so the serial chain has
// no division and no power of z overflows.
template <typename T>
__device__ inline void leaf_bessel(const LeafNode<T> &d, int p, int N, const cx<T> *inv, cx<T> *out, int stride) {
    const cx<T> z2 = d.z * d.z;
    cx<T> g1 = d.g1, g = d.g0;                          // g_{n+1}, g_n
#pragma unroll 4
    for (int n = p; n >= 1; --n) {
        if (n <= N) out[n * stride] = g;
        const cx<T> h = g - (inv[n].im * z2) * g1;
        g1 = g;
        g = h;
    }
    out[0] = g;
    cx<T> pw = mk(T(1), T(0));
#pragma unroll 4
    for (int n = 1; n <= N; ++n) {
        pw = (inv[n].re * d.z) * pw;
        out[n * stride] = pw * out[n * stride];
    }
}

// Rows of a local expansion's coefficients for leaf_eval, [(n, m, cos | sin)][CW]:
// row n (n + 1) + 2 m + (sin) of degree n, order m.  a multiplies R_n^m and b R_n^{-m}.
template <typename T>
__device__ __forceinline__ void leaf_rows(cx<T> *row, int half, int m, cx<T> a, cx<T> b) {
    row[0] = m ? a + b : a;
    row[half] = m ? mk(b.im - a.im, a.re - b.re) : mk(T(0), T(0));   // i (a - b)
}

// (la, lb) of degrees <= N side by side in LDS, row stride S, with one row's slack
template <typename T>
__device__ inline void leaf_tables(const BasisTab<T> &bt, int N, cx<T> *lab, T *qs) {
    const int S = bt.N + 1;
    for (int t = threadIdx.x; t < (N + 1) * S; t += blockDim.x) lab[t] = mk(bt.la[t], bt.lb[t]);
    for (int t = threadIdx.x; t < S; t += blockDim.x) {
        lab[(N + 1) * S + t] = mk(T(0), T(0));
        qs[t] = (t & 1) ? -bt.qmm[t] : bt.qmm[t];
    }
}

// One wavefront: values at 16 nodes (rows, node l % 16 of lane l) of the CW / 2 <= 8
// complex expansions in rows[], degrees <= N < 2 TT.  x, w: the lane's node's direction;
// J[n * JS + i] = j_n of the tile's node i.  Register q of lane l is column l % 16 of node
// row(l / 16, q).  Each degree's sum over orders is one chain of n / 2 + 1 steps;
// j_n, complex for lossy media, multiplies its 16 x 16 result.
template <typename T, int TT>
__device__ inline typename Mma16<T>::v4 leaf_eval(const T *rows, int CW, const cx<T> *lab, int S, const T *qs, int N,
                                                  T x, cx<T> w, const cx<T> *J, int JS) {
    typedef typename Mma16<T>::v4 v4;
    const int lane = threadIdx.x & 63, col = lane & 15, kq = lane >> 4, ms = kq >> 1;
    const T *row = rows + kq * CW + (col < CW ? col : 0);
    T q1[TT], q2[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) q1[t] = q2[t] = T(0);
    cx<T> wn = mk(T(1), T(0));
    v4 aR = {0, 0, 0, 0}, aI = {0, 0, 0, 0};
    for (int n = 0; n <= N; ++n) {
        if (n) wn = wn * w;
        const T st = qs[n] * ((kq & 1) ? wn.im : wn.re);
        v4 z = {0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < TT; ++t)
            if (2 * t <= n) {
                const int m = 2 * t + ms;
                const cx<T> ab = lab[n * S + m];
                T v = ab.re * (x * q1[t] - ab.im * q2[t]);
                if (2 * t + 1 >= n) v = m == n ? st : (m > n ? T(0) : v);
                q2[t] = q1[t];
                q1[t] = v;
                z = Mma16<T>::mma(v, row[4 * t * CW], z);
            }
        row += 2 * (n + 1) * CW;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const cx<T> j = J[n * JS + Mma16<T>::row(kq, q)];
            aR[q] += j.re * z[q];
            aI[q] += j.im * z[q];
        }
    }
    v4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const T s = lane_swap(aI[q]);
        o[q] = (col & 1) ? aR[q] + s : aR[q] - s;
    }
    return o;
}

}  // namespace fmb
