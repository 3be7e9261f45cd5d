// One fast-multipole matvec y = Op_k(a, b) (Sec. 2.2, Steps 1-4).
//
// Each output channel c = x, y, z is a Helmholtz potential of sources that
// carry a monopole and a dipole:
//   y_c(s_alpha) = sum_beta [ sigma_{beta,c} g(s_beta, s_alpha) + q_{beta,c} . grad' g(s_beta, s_alpha) ],
//   sigma_{beta,c} = w b_c,   q_{beta,c} = w (n_c a - a_c n - (n . a) e_c),
// which is the kernel n (grad'g . a) - (n . grad'g) a - grad'g (n . a) + g b of
// eq. 2.12 written per component.  Hence
//   Step 1 (eqs. 2.18-2.19): M_nm,c = i k sum_beta [sigma_c R_n^-m + q_c . grad R_n^-m](s_beta - X),
//   Step 2 (eq. 2.20): S|S to the parent, Step 3 (eq. 2.21): S|R over FF plus
//   R|R from the parent, Step 4 (eq. 2.23): y_c = sum L_nm,c R_n^m(s - X) plus
//   the near sum over the leaf and its neighbours.
// Gradients of R_n^m use the recurrences that follow from the plane-wave form
// of R (cos(theta) and sin(theta) e^{+-i phi} times Y_n^m shift n by one):
//   d_z R_n^m        = k [ -A_n^m R_{n+1}^m     + B_n^m R_{n-1}^m ]
//   (d_x + i d_y) R  = k [ -C_n^m R_{n+1}^{m+1} + D_n^m R_{n-1}^{m+1} ]
//   (d_x - i d_y) R  = k [ -E_n^m R_{n+1}^{m-1} + F_n^m R_{n-1}^{m-1} ]
#include <array>
#include <map>

#include "basis.h"
#include "plan.h"

namespace fmb {

namespace {

constexpr int TPB = 256;

// ---------------------------------------------------------------- gather
template <typename T>
__global__ void k_gather_src(const cx<T> *__restrict__ a, const cx<T> *__restrict__ b, const int32_t *__restrict__ perm,
                             const double *__restrict__ sw, const double *__restrict__ snrm, int64_t n, int nrhs,
                             cx<T> *__restrict__ src) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    const T w = (T)sw[i];
    const T nx = (T)snrm[3 * i], ny = (T)snrm[3 * i + 1], nz = (T)snrm[3 * i + 2];
    for (int r = 0; r < nrhs; ++r) {
        const cx<T> *A = a + ((int64_t)r * n + u) * 3;
        const cx<T> *B = b + ((int64_t)r * n + u) * 3;
        cx<T> *o = src + ((int64_t)r * n + i) * 7;
        cx<T> wa0 = w * A[0], wa1 = w * A[1], wa2 = w * A[2];
        o[0] = wa0;
        o[1] = wa1;
        o[2] = wa2;
        o[3] = w * B[0];
        o[4] = w * B[1];
        o[5] = w * B[2];
        o[6] = nx * wa0 + ny * wa1 + nz * wa2;
    }
}

template <typename T>
__global__ void k_scatter_out(const cx<T> *__restrict__ ys, const int32_t *__restrict__ perm, int64_t n, int nrhs,
                              cx<T> *__restrict__ y) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    for (int r = 0; r < nrhs; ++r)
        for (int c = 0; c < 3; ++c) y[((int64_t)r * n + u) * 3 + c] = ys[((int64_t)r * n + i) * 3 + c];
}

// MI355X dispatches consecutive workgroups to its 8 XCDs in turn.  Tiles are
// listed operator by operator; renumbering block i to tile (i % 8) * chunk + i / 8
// gives each XCD a contiguous run of tiles, so the tiles that share an operator
// share one L2.  The grid is padded to a multiple of 8; spare blocks exit.
__device__ inline int xcd_tile(int i, int ntiles) {
    const int chunk = (ntiles + 7) / 8;
    return (i % 8) * chunk + i / 8;
}

// ---------------------------------------------------------------- P2M
// One block per leaf and right-hand side, NG groups of 4 nodes at a time.  With W = n x a
// the dipole part n (a . g) - a (n . g) - (n . a) g of a node is g x W - (n . a) g, so the
// multipoles follow from the moments of seven complex densities (W, n . a, b) with
// R_n^m, n <= p, and one gradient recurrence per coefficient instead of one per
// coefficient and node.  The moments are a product on the matrix cores: wavefront t
// owns the orders m = 8 t .. 8 t + 7 (16 rows: cos and sin), the columns are re and im
// of the densities times j_n, the nodes are summed over.  The block walks the
// degrees together: moments of degree n go to a ring of four degrees in LDS, then
// the multipoles of degree n - 1 are formed from degrees n - 2 .. n:
//   d_z = c0 Q[n+1, mu] + c1 Q[n-1, mu],  d_+- = c2|c4 Q[n+1, mu +- 1] + c3|c5 Q[n-1, mu +- 1],
//   grad = k ((d_+ + d_-) / 2, (d_+ - d_-) / 2i, d_z),  mu = -m.
// Leaves of more than 4 NG nodes add chunk by chunk.  Bound by latency: the degrees are a
// serial chain of a short product, a barrier and a gradient step (a branch and its LDS latency per
// group of 4 nodes cost 3/4 of the time before GS groups were loaded together).  One thread per
// coefficient, gathering six table entries per node, took 5.7 ms for 753k nodes at order 17
// in FP64 and 0.81 ms for 60k at 23, now 1.74 and 0.27; 4.2 ms for 3M at 12 in FP32, now 1.75.
template <typename T, int NG>
__global__ void __launch_bounds__(384, sizeof(T) == 8 ? 2 : (NG == 16 ? 3 : 4))
    k_p2m(const int32_t *__restrict__ start, const LeafNode<T> *__restrict__ geo, const double *__restrict__ snrm,
          const cx<T> *__restrict__ src, int64_t n, int p, double k_re, double k_im, const double *__restrict__ inv_alpha,
          const T *__restrict__ tab, int nrhs_max, cx<T> *__restrict__ M) {
    typedef typename Mma16<T>::v4 v4;
    extern __shared__ unsigned char smem[];
    constexpr int NB = 4 * NG, GS = NG / 4;     // GS groups' loads ahead of their products
    const int N = p, P2 = p * p, W2 = 2 * N + 1;
    const BasisTab<T> bt = basis_tab(tab, N);
    cx<T> *J = reinterpret_cast<cx<T> *>(smem);                         // [N+1][NB]
    cx<T> *inv = J + (N + 1) * NB;                                      // [N+1]
    cx<T> *sc = inv + N + 1;                                            // [p] i k / alpha_n
    cx<T> *lab = sc + p;                                                // [N+1][N+1] la, lb (zero up to the diagonal)
    T *V = reinterpret_cast<T *>(lab + (N + 1) * (N + 1));              // [NB][16] densities
    T *xs = V + NB * 16;                                                // [NB] cos th
    cx<T> *wp = reinterpret_cast<cx<T> *>(xs + NB);                     // [N+1][NB] powers of sin th e^{i ph}, then
    cx<T> *ring = wp;                                                   // [4][W2][7] moments of four degrees
    const int box = blockIdx.x, r = blockIdx.y;
    const int s0 = start[box], s1 = start[box + 1];
    const cx<T> k = mk((T)k_re, (T)k_im);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int kq = lane >> 4, col = lane & 15;
    // the lane's row as input (order, cos | sin)
    const int rq = Mma16<T>::q_of(col), rm = 8 * wave + 2 * Mma16<T>::kq_of(col) + (rq >> 1);
    const int mc = min(rm, N);
    const bool sine = rq & 1;
    leaf_inv_table(N, inv);
    for (int t = threadIdx.x; t < (N + 1) * (N + 1); t += blockDim.x) lab[t] = mk(bt.la[t], bt.lb[t]);
    for (int t = threadIdx.x; t < p; t += blockDim.x) sc[t] = mk((T)(-k_im * inv_alpha[t]), (T)(k_re * inv_alpha[t]));
    cx<T> *Mo = M + ((int64_t)box * nrhs_max + r) * 3 * P2;
    if (s0 == s1)
        for (int t = threadIdx.x; t < 3 * P2; t += blockDim.x) Mo[t] = mk(T(0), T(0));
    for (int b0 = s0; b0 < s1; b0 += NB) {
        const int nb = min(NB, s1 - b0);
        leaf_sync();
        for (int t = threadIdx.x; t < 2 * NB; t += blockDim.x) {
            const int j = t % NB;
            const int64_t i = b0 + min(j, nb - 1);
            const LeafNode<T> d = geo[i];
            if (t < NB) {
                leaf_bessel(d, N, N, inv, J + j, NB);
                continue;
            }
            xs[j] = d.x;
            cx<T> wm = mk(T(1), T(0));
            for (int m = 0; m <= N; ++m) {
                wp[m * NB + j] = wm;
                wm = wm * d.w;
            }
            cx<T> v[8];
            for (int q = 0; q < 8; ++q) v[q] = mk(T(0), T(0));
            if (j < nb) {
                const cx<T> *sr = src + ((int64_t)r * n + i) * 7;
                const T nv[3] = {(T)snrm[3 * i], (T)snrm[3 * i + 1], (T)snrm[3 * i + 2]};
                const cx<T> a[3] = {sr[0], sr[1], sr[2]};
                for (int c = 0; c < 3; ++c) {
                    v[c] = nv[(c + 1) % 3] * a[(c + 2) % 3] - nv[(c + 2) % 3] * a[(c + 1) % 3];
                    v[4 + c] = sr[3 + c];
                }
                v[3] = sr[6];
            }
            for (int q = 0; q < 8; ++q) *reinterpret_cast<cx<T> *>(V + j * 16 + 2 * q) = v[q];
        }
        leaf_sync();
        // a lane holds its first value until degree m (rows of orders above the degree are not read)
        T q1[NG], q2[NG], x[NG], v0[NG];
        const T qs = (rm > N ? T(0) : T(1)) * ((mc & 1) ? -bt.qmm[mc] : bt.qmm[mc]);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int j = 4 * g + kq;
            const cx<T> wm = wp[mc * NB + j];
            q1[g] = qs * (sine ? wm.im : wm.re);
            q2[g] = T(0);
            x[g] = xs[j];
            v0[g] = V[j * 16 + col];
        }
        leaf_sync();
        for (int nn = 0; nn <= N; ++nn) {
            const int nm = nn - 1;
            // gradient coefficients of the multipoles formed below: loaded ahead of the products
            T co[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) co[q] = bt.gco[min(max(nm, 0) * max(nm, 0) + lane, P2 - 1) * 6 + q];
            cx<T> *rg = ring + (nn & 3) * 7 * W2;
            // orders up to two beyond the degree are written as zeros: the recurrences read them
            if (8 * wave <= nn + 2) {
                const T la = lab[nn * (N + 1) + mc].re, lb = lab[nn * (N + 1) + mc].im;
                const T hold = nn <= mc ? T(1) : T(0), neg = (col & 1) ? T(1) : T(-1);
                const cx<T> *Jn = J + nn * NB + kq;
                v4 acc = {0, 0, 0, 0}, acc2 = acc;
                if (8 * wave <= nn) {
#pragma unroll
                    for (int g0 = 0; g0 < NG; g0 += GS)
                        if (4 * g0 < nb) {
                            cx<T> j[GS];
#pragma unroll
                            for (int g = 0; g < GS; ++g) j[g] = Jn[4 * (g0 + g)];
#pragma unroll
                            for (int g = 0; g < GS; ++g) {
                                const T u = la * (x[g0 + g] * q1[g0 + g] - lb * q2[g0 + g]) + hold * q1[g0 + g];
                                q2[g0 + g] = q1[g0 + g];
                                q1[g0 + g] = u;
                                const T d = j[g].re * v0[g0 + g] + (neg * j[g].im) * lane_swap(v0[g0 + g]);
                                if (g & 1) acc2 = Mma16<T>::mma(u, d, acc2);
                                else acc = Mma16<T>::mma(u, d, acc);
                            }
                        }
                    acc += acc2;
                }
                // registers (0, 1) and (2, 3) are cos and sin of two orders
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int m = 8 * wave + 2 * kq + h;
                    const T o = lane_swap(acc[2 * h + 1]), s = (col & 1) ? o : -o;
                    if (m <= min(nn + 2, N) && col < 14) {
                        T *at = reinterpret_cast<T *>(rg + 7 * N) + col;
                        at[14 * m] = m <= nn ? acc[2 * h] + s : T(0);
                        if (m) at[-14 * m] = m <= nn ? acc[2 * h] - s : T(0);
                    }
                }
            }
            leaf_sync();
            if (nm < 0) continue;
            // (degree -1 has zero coefficients: any finite values serve)
            const cx<T> *up0 = rg + 7 * N, *dn0 = (nm ? ring + ((nn + 2) & 3) * 7 * W2 : rg) + 7 * N;
            const cx<T> *mid0 = ring + ((nn + 3) & 3) * 7 * W2 + 7 * N;
            for (int e = lane; e <= 2 * nm; e += 64) {
                const int mu = nm - e, idx = nm * nm + e;
                if (e >= 64)
#pragma unroll
                    for (int q = 0; q < 6; ++q) co[q] = bt.gco[idx * 6 + q];
                const cx<T> *up = up0 + 7 * mu, *dn = dn0 + 7 * mu;
                auto dz = [&](int v) { return co[0] * up[v] + co[1] * dn[v]; };
                auto dp = [&](int v) { return co[2] * up[7 + v] + co[3] * dn[7 + v]; };
                auto dm = [&](int v) { return co[4] * up[v - 7] + co[5] * dn[v - 7]; };
                auto dx = [&](int v) { return T(0.5) * (dp(v) + dm(v)); };
                auto dy = [&](int v) {
                    const cx<T> df = dp(v) - dm(v);
                    return mk(T(0.5) * df.im, T(-0.5) * df.re);
                };
                for (int c = wave; c < 3; c += nw) {
                    cx<T> gr;
                    if (c == 0) gr = dy(2) - dz(1) - dx(3);
                    else if (c == 1) gr = dz(0) - dx(2) - dy(3);
                    else gr = dx(1) - dy(0) - dz(3);
                    const cx<T> m = sc[nm] * (mid0[7 * mu + 4 + c] + k * gr);
                    cx<T> *o = Mo + c * P2 + idx;
                    *o = b0 == s0 ? m : *o + m;
                }
            }
        }
    }
}

template <typename T, int NG>
size_t p2m_lds(int N) {
    return ((size_t)(N + 1) * 4 * NG + 2 * N + 1 + (size_t)(N + 1) * (N + 1)) * sizeof(cx<T>) +
           (size_t)4 * NG * 17 * sizeof(T) +
           std::max((size_t)(N + 1) * 4 * NG, (size_t)28 * (2 * N + 1)) * sizeof(cx<T>);
}

// Chunks of 64 nodes instead of 32, where two blocks' tables fit a CU: when a leaf has more than 32 on average, or when
// some leaf has and the grid is short, so that the fullest leaves' second chunk would be waited for.  Short: two rounds
// of what the CUs hold by LDS (eight blocks at most), for the plan's largest batch, so that a column's sums do not depend
// on how many there are.  Chunks of 32 / 64, fullest leaf 40 or 59 (us): 532 leaves FP32 p = 5 31 / 21, FP64 p = 16
// 66 / 58; 2,320 leaves FP32 p = 5 36 / 27, FP64 p = 16 156 / 178; 4,256 blocks FP64 p = 16 207 / 280.
template <typename T>
bool p2m_wide(const Plan &P) {
    const size_t lds = p2m_lds<T, 16>(P.order);
    const int64_t nbox = P.lv[P.depth].nbox;
    if (lds > 80 * 1024) return false;
    return P.n > 32 * nbox ||
           (P.leaf_max > 32 && nbox * P.nrhs_max <= 512 * (int64_t)std::min<size_t>(8, LEAF_LDS_MAX / lds));
}

// ---------------------------------------------------------------- L2P
// One block per leaf and RC right-hand sides, 16 nodes per wavefront at a time: the
// coefficients are laid out once per block as the rows that leaf_eval multiplies
// (6 RC of 16 columns: re and im of three channels), j_n of 16 nodes per wavefront
// and the recurrence constants beside them.  One lane per node took 1.3 ms for 753k nodes at order 17
// in FP64 and 0.52 ms for 60k at 23, now 0.56 and 0.17; loading two or four steps ahead does
// work for absent orders and was slower (0.58, 0.80 ms).
template <typename T, int RC, int TT>
__global__ void __launch_bounds__(256) k_l2p(const int32_t *__restrict__ start, const LeafNode<T> *__restrict__ geo,
                                            int64_t n, int p, const double *__restrict__ inv_alpha,
                                            const T *__restrict__ tab, int nrhs, int nrhs_max,
                                            const cx<T> *__restrict__ Lc, cx<T> *__restrict__ ys) {
    extern __shared__ unsigned char smem[];
    constexpr int CW = 6 * RC;
    const int P2 = p * p, N = p - 1, S = p + 1, NB = blockDim.x / 4;
    const BasisTab<T> bt = basis_tab(tab, p);
    cx<T> *inv = reinterpret_cast<cx<T> *>(smem);                       // [p+1]
    cx<T> *lab = inv + p + 1;                                           // [p+1][S]
    cx<T> *J = lab + (p + 1) * S;                                       // [p][NB]
    cx<T> *rows = J + p * NB;                                           // [p (p+1) + 2][CW / 2]
    T *qs = reinterpret_cast<T *>(rows + (p * (p + 1) + 2) * (CW / 2)); // [S]
    const int box = blockIdx.x, r0 = blockIdx.y * RC;
    const int rcn = min(RC, nrhs - r0);
    const int s0 = start[box], s1 = start[box + 1];
    leaf_inv_table(p, inv);
    leaf_tables(bt, N, lab, qs);
    for (int t = threadIdx.x; t < 2 * (CW / 2); t += blockDim.x) rows[p * (p + 1) * (CW / 2) + t] = mk(T(0), T(0));
    for (int idx = threadIdx.x; idx < P2; idx += blockDim.x) {
        int nn = (int)sqrtf((float)idx);
        if (nn * nn > idx) --nn;
        if ((nn + 1) * (nn + 1) <= idx) ++nn;
        const int m = idx - nn * nn - nn;
        if (m < 0) continue;
        const T ia = (T)inv_alpha[nn];
        cx<T> *o = rows + (nn * (nn + 1) + 2 * m) * (CW / 2);
        for (int e = 0; e < 3 * RC; ++e) {
            cx<T> a = mk(T(0), T(0)), b = a;
            if (e / 3 < rcn) {
                const cx<T> *L = Lc + (((int64_t)box * nrhs_max + r0) * 3 + e) * P2 + idx;
                a = ia * L[0];
                b = ia * L[-2 * m];
            }
            leaf_rows(o + e, CW / 2, m, a, b);
        }
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, kq = lane >> 4;
    for (int b0 = s0; b0 < s1; b0 += NB) {
        leaf_sync();
        if ((int)threadIdx.x < NB)
            leaf_bessel(geo[min(b0 + (int)threadIdx.x, s1 - 1)], p, N, inv, J + threadIdx.x, NB);
        leaf_sync();
        const int t0 = b0 + 16 * wave;
        if (t0 >= s1) continue;
        const LeafNode<T> d = geo[min(t0 + col, s1 - 1)];
        const auto o = leaf_eval<T, TT>(reinterpret_cast<const T *>(rows), CW, lab, S, qs, N, d.x, d.w, J + 16 * wave, NB);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = t0 + Mma16<T>::row(kq, q);
            if (i < s1 && col < 6 * rcn)
                reinterpret_cast<T *>(ys + ((int64_t)(r0 + col / 6) * n + i) * 3)[col % 6] = o[q];
        }
    }
}

// LDS of k_l2p for RC right-hand sides a block
template <typename T>
size_t l2p_lds(int p, int rc, int waves) {
    return (p + 1) * sizeof(T) +
           ((size_t)(p + 1) * (p + 2) + (size_t)p * 16 * waves + (size_t)(p * (p + 1) + 2) * 3 * rc) * sizeof(cx<T>);
}

// Two right-hand sides a block share the recurrence; one at a time where two do not fit a block's LDS (FP64 leaf
// orders from 34 with four wavefronts, 37 with one; one fits at every order: 147 KB at 40).
template <typename T>
void launch_l2p(Plan &P, int nrhs, const cx<T> *Lc, cx<T> *ys, hipStream_t s) {
    const int p = P.order;
    const Level &LL = P.lv[P.depth];
    // wavefronts for the nodes of an average leaf
    const int waves = (int)std::min<int64_t>(4, std::max<int64_t>(1, (P.n + 16 * LL.nbox - 1) / (16 * LL.nbox)));
    const int rc = nrhs > 1 && l2p_lds<T>(p, 2, waves) <= LEAF_LDS_MAX ? 2 : 1;
    const size_t sh = l2p_lds<T>(p, rc, waves);
    auto of = [&](auto k8, auto k16, auto k24, auto k40) { return p <= 8 ? k8 : (p <= 16 ? k16 : (p <= 24 ? k24 : k40)); };
    auto kern = rc == 2 ? of(k_l2p<T, 2, 4>, k_l2p<T, 2, 8>, k_l2p<T, 2, 12>, k_l2p<T, 2, 20>)
                        : of(k_l2p<T, 1, 4>, k_l2p<T, 1, 8>, k_l2p<T, 1, 12>, k_l2p<T, 1, 20>);
    leaf_lds_limit(kern, sh);
    kern<<<dim3((unsigned)LL.nbox, (unsigned)((nrhs + rc - 1) / rc)), 64 * waves, sh, s>>>(
        LL.start.as<int32_t>(), P.lnode.as<LeafNode<T>>(), P.n, p, P.inv_alpha.as<double>() + (size_t)P.depth * p,
        P.btab.as<T>(), nrhs, P.nrhs_max, Lc, ys);
    FMB_LAUNCH_CHECK();
}

// ---------------------------------------------------------------- P2P
// FP64 near field, one block per leaf.  Targets on lanes; when a leaf holds fewer targets
// than the block has threads, the sources are split into S slices handled by
// the spare threads and the slices are summed in LDS at the end.  A source's dipole part
// n (d . a) - a (d . n) - d (n . a) is d x W - d (n . a) with W = n x a formed once per
// source as it is staged.  The kernel is bound by its FP64 arithmetic (about 110 instructions a
// pair with real k, a quarter of them the sine and cosine); the source tile is small enough for
// four wavefronts a SIMD.  148k-node ring 1.83 -> 1.21 ms against library sine, root and division, normals
// in the tile and two wavefronts a SIMD; 753k-node ellipsoid 6.56 -> 4.25 ms.
constexpr int P2P_TILE = 128;

struct alignas(16) Src64 {
    double x, y, z;
    int32_t tri, pad;
    cx<double> w[3], na, b[3];
};

template <bool LOSSY>
__global__ void __launch_bounds__(TPB, 4)
    k_p2p64(const int32_t *__restrict__ start, const int32_t *__restrict__ nbr, const double *__restrict__ spts,
            const double *__restrict__ snrm, const int32_t *__restrict__ stri, const cx<double> *__restrict__ src, int64_t n,
            double kr, double ki, double rcut2, cx<double> *__restrict__ ys) {
    __shared__ union {
        Src64 tile[P2P_TILE];
        cx<double> red[TPB][3];
    } sh;
    __shared__ int32_t nb_start[28], nb_box[27];
    __shared__ int n_nb;
    const int box = blockIdx.x, r = blockIdx.y;
    const int t0 = start[box], t1 = start[box + 1];
    const int nt = t1 - t0;
    if (threadIdx.x == 0) {
        int c = 0, tot = 0;
        for (int s = 0; s < 27; ++s) {
            int q = nbr[box * 27 + s];
            if (q >= 0) {
                nb_box[c] = q;
                nb_start[c] = tot;
                tot += start[q + 1] - start[q];
                ++c;
            }
        }
        nb_start[c] = tot;
        n_nb = c;
    }
    __syncthreads();
    const int ns_total = nb_start[n_nb];
    const double inv4pi = 0.07957747154594766788;
    for (int tc0 = 0; tc0 < nt; tc0 += TPB) {
        const int ntc = min(TPB, nt - tc0);
        const int S = TPB / ntc;                 // source slices
        const int ti = threadIdx.x % ntc, sl = threadIdx.x / ntc;
        const bool active = sl < S;
        double tp[3] = {0, 0, 0};
        int32_t ttri = -1;
        if (active) {
            const int64_t ig = t0 + tc0 + ti;
            for (int q = 0; q < 3; ++q) tp[q] = spts[3 * ig + q];
            ttri = stri[ig];
        }
        cx<double> acc[3] = {mk(0.0, 0.0), mk(0.0, 0.0), mk(0.0, 0.0)};
        for (int base = 0; base < ns_total; base += P2P_TILE) {
            const int cnt = min(P2P_TILE, ns_total - base);
            __syncthreads();
            for (int j = threadIdx.x; j < cnt; j += blockDim.x) {
                const int u = base + j;
                int b = 0;
                while (nb_start[b + 1] <= u) ++b;
                const int64_t sidx = start[nb_box[b]] + (u - nb_start[b]);
                const cx<double> *sr = src + ((int64_t)r * n + sidx) * 7;
                const cx<double> a[3] = {sr[0], sr[1], sr[2]};
                Src64 o;
                o.x = spts[3 * sidx];
                o.y = spts[3 * sidx + 1];
                o.z = spts[3 * sidx + 2];
                o.tri = stri[sidx];
                o.pad = 0;
                const double nv[3] = {snrm[3 * sidx], snrm[3 * sidx + 1], snrm[3 * sidx + 2]};
                for (int c = 0; c < 3; ++c) {
                    o.w[c] = nv[(c + 1) % 3] * a[(c + 2) % 3] - nv[(c + 2) % 3] * a[(c + 1) % 3];
                    o.b[c] = sr[3 + c];
                }
                o.na = sr[6];
                sh.tile[j] = o;
            }
            __syncthreads();
            if (!active) continue;
            for (int j = sl; j < cnt; j += S) {
                const Src64 &o = sh.tile[j];
                if (o.tri == ttri) continue;
                const double dx = o.x - tp[0], dy = o.y - tp[1], dz = o.z - tp[2];
                const double R2 = dx * dx + dy * dy + dz * dz;
                if (R2 > rcut2) continue;       // damped below the cutoff (local-only lossy plans)
                const double iR = fast_rsqrt(R2), R = R2 * iR;
                double sn, cs;
                fast_sincos(kr * R, &sn, &cs);
                double h = inv4pi * iR;
                if (LOSSY) h *= fast_exp(-ki * R);
                const cx<double> g = mk(h * cs, h * sn);
                // f = (i k R - 1) g / R^2
                const double i2 = iR * iR, fr = LOSSY ? -(ki * R + 1.0) * i2 : -i2, fi = kr * iR;
                const cx<double> f = mk(fr * g.re - fi * g.im, fr * g.im + fi * g.re);
                acc[0] += f * (dy * o.w[2] - dz * o.w[1] - dx * o.na) + g * o.b[0];
                acc[1] += f * (dz * o.w[0] - dx * o.w[2] - dy * o.na) + g * o.b[1];
                acc[2] += f * (dx * o.w[1] - dy * o.w[0] - dz * o.na) + g * o.b[2];
            }
        }
        __syncthreads();
        for (int c = 0; c < 3; ++c) sh.red[threadIdx.x][c] = acc[c];
        __syncthreads();
        if (threadIdx.x < ntc) {
            cx<double> s[3] = {mk(0.0, 0.0), mk(0.0, 0.0), mk(0.0, 0.0)};
            for (int q = 0; q < S; ++q)
                for (int c = 0; c < 3; ++c) s[c] += sh.red[q * ntc + threadIdx.x][c];
            cx<double> *o = ys + ((int64_t)r * n + t0 + tc0 + threadIdx.x) * 3;
            for (int c = 0; c < 3; ++c) o[c] += s[c];
        }
        __syncthreads();
    }
}

// FP32 near field, one block per leaf in Morton order.  Consecutive blocks go
// to different XCDs; giving each XCD contiguous runs of leaves cuts the L2-miss
// traffic (52 -> 12 MB per launch on the 60k-node torus) but unbalances the
// load and is slower, and the kernel is bound by its arithmetic.  Source
// records are packed into five 16-byte LDS words per source: position relative
// to the target leaf's centre (FP32; the leaf and its neighbours span a few
// leaf widths, so the difference keeps FP32 relative accuracy) with the
// triangle id, and seven density values: W = n x a formed once per source (the
// dipole part n (d . a) - a (d . n) - d (n . a) is d x W - d (n . a)), b and n . a.  The transcendentals
// go straight to the hardware units with the scale folded into the constants:
// v_sin/v_cos take revolutions (kR / 2 pi), v_exp takes a base-2 exponent
// (-Im k R log2 e); the LOSSY = false instance (real k) skips the decay
// factor.  Same-triangle pairs are masked, not branched around, so the source
// loop unrolls.
struct __attribute__((aligned(16))) SrcHdr32 {
    float x, y, z;
    int32_t tri;
    float nx, ny, nz, pad;
};

// RC right-hand sides per block (blockIdx.y = chunk of RC): the pair geometry,
// the transcendentals and g, f are computed once per pair and applied to all
// RC density sets.  The source tile shrinks as RC grows to keep LDS near 32 KB.
// word pair w of a staged record: (W_w, b_w) for w < 3, n . a for w = 3
__device__ __forceinline__ void stage_rec32(const SrcHdr32 &h, const cx<float> *__restrict__ sr, int w, cx<float> *rec) {
    if (w == 3) {
        rec[6] = sr[6];
        return;
    }
    const int u = w == 2 ? 0 : w + 1, v = w == 0 ? 2 : w - 1;
    const float n1 = w == 0 ? h.ny : (w == 1 ? h.nz : h.nx), n2 = w == 0 ? h.nz : (w == 1 ? h.nx : h.ny);
    rec[w] = n1 * sr[v] - n2 * sr[u];
    rec[3 + w] = sr[3 + w];
}

template <int RC>
struct P2PTile {
    static constexpr int TS = RC == 1 ? 256 : (RC == 2 ? 128 : 64);
};

template <bool LOSSY, int RC, bool CUT = false>
__global__ void __launch_bounds__(TPB) k_p2p32(int nleaf, int nrhs, const int32_t *__restrict__ start,
                                               const int32_t *__restrict__ nbr,
                                               const double *__restrict__ center, const double *__restrict__ spts,
                                               const double *__restrict__ snrm, const int32_t *__restrict__ stri,
                                               const cx<float> *__restrict__ src, int64_t n, double k_re,
                                               double k_im, float rcut2, cx<float> *__restrict__ ys) {
    constexpr int TS = P2PTile<RC>::TS;
    __shared__ SrcHdr32 hdr[TS];
    __shared__ __attribute__((aligned(16))) cx<float> rec[TS][RC][8];   // n x a, b, n.a, unused
    __shared__ int32_t sid[TS];
    __shared__ int32_t nb_start[28], nb_box[27];
    __shared__ int n_nb;
    __shared__ cx<float> red[TPB][3];
    const int box = blockIdx.x, r0 = blockIdx.y * RC;
    if (box >= nleaf) return;
    const int rcn = min(RC, nrhs - r0);
    const int t0 = start[box], t1 = start[box + 1];
    const int nt = t1 - t0;
    const double c0x = center[3 * box], c0y = center[3 * box + 1], c0z = center[3 * box + 2];
    if (threadIdx.x == 0) {
        int c = 0, tot = 0;
        for (int s = 0; s < 27; ++s) {
            int q = nbr[box * 27 + s];
            if (q >= 0) {
                nb_box[c] = q;
                nb_start[c] = tot;
                tot += start[q + 1] - start[q];
                ++c;
            }
        }
        nb_start[c] = tot;
        n_nb = c;
    }
    __syncthreads();
    const int ns_total = nb_start[n_nb];
    const float krev = (float)(k_re * 0.15915494309189533577);        // k_re / (2 pi)
    const float kexp = (float)(-k_im * 1.44269504088896340736);       // -k_im log2(e)
    const float kr = (float)k_re, ki = (float)k_im;
    const float inv4pi = 0.07957747154594766788f;
    for (int tc0 = 0; tc0 < nt; tc0 += TPB) {
        const int ntc = min(TPB, nt - tc0);
        const int S = TPB / ntc;
        const int ti = threadIdx.x % ntc, sl = threadIdx.x / ntc;
        const bool active = sl < S;
        const int64_t ig = t0 + tc0 + ti;
        float tx = 0.f, ty = 0.f, tz = 0.f;
        int32_t ttri = -1;
        if (active) {
            tx = (float)(spts[3 * ig] - c0x);
            ty = (float)(spts[3 * ig + 1] - c0y);
            tz = (float)(spts[3 * ig + 2] - c0z);
            ttri = stri[ig];
        }
        cx<float> acc[RC][3];
#pragma unroll
        for (int rr = 0; rr < RC; ++rr)
            for (int c = 0; c < 3; ++c) acc[rr][c] = mk(0.f, 0.f);
        for (int base = 0; base < ns_total; base += TS) {
            const int cnt = min(TS, ns_total - base);
            __syncthreads();
            for (int j = threadIdx.x; j < cnt; j += blockDim.x) {
                const int u = base + j;
                int b = 0;
                while (nb_start[b + 1] <= u) ++b;
                const int64_t sidx = start[nb_box[b]] + (u - nb_start[b]);
                SrcHdr32 q;
                q.x = (float)(spts[3 * sidx] - c0x);
                q.y = (float)(spts[3 * sidx + 1] - c0y);
                q.z = (float)(spts[3 * sidx + 2] - c0z);
                q.tri = stri[sidx];
                q.nx = (float)snrm[3 * sidx];
                q.ny = (float)snrm[3 * sidx + 1];
                q.nz = (float)snrm[3 * sidx + 2];
                q.pad = 0.f;
                hdr[j] = q;
                sid[j] = (int32_t)sidx;
            }
            __syncthreads();
            for (int e = threadIdx.x; e < cnt * RC * 4; e += blockDim.x) {
                const int rr = (e / 4) % RC, j = e / (4 * RC);
                // chunks beyond the last right-hand side repeat it (their sums are not written)
                stage_rec32(hdr[j], src + ((int64_t)(r0 + min(rr, rcn - 1)) * n + sid[j]) * 7, e % 4, rec[j][rr]);
            }
            __syncthreads();
            if (!active) continue;
#pragma unroll 2
            for (int j = sl; j < cnt; j += S) {
                const SrcHdr32 &q = hdr[j];
                const bool self = q.tri == ttri;
                const float dx = q.x - tx, dy = q.y - ty, dz = q.z - tz;
                if (CUT && dx * dx + dy * dy + dz * dz > rcut2) continue;   // damped below the cutoff
                const float R2 = self ? 1.f : dx * dx + dy * dy + dz * dz;
                const float iR = __builtin_amdgcn_rsqf(R2);
                const float R = R2 * iR;
                const float sn = __builtin_amdgcn_sinf(krev * R), cs = __builtin_amdgcn_cosf(krev * R);
                const float ex = LOSSY ? __builtin_amdgcn_exp2f(kexp * R) : 1.f;   // real k: no decay
                const float sc = self ? 0.f : inv4pi * iR * ex;            // e^{-Im k R} / (4 pi R)
                const cx<float> g = mk(sc * cs, sc * sn);                   // e^{ikR} / (4 pi R)
                const float iR2 = iR * iR;
                // f = (i k R - 1) g / R^2
                const float fr = LOSSY ? iR2 * (-ki * R - 1.f) : -iR2, fi = kr * iR;
                const cx<float> f = mk(fr * g.re - fi * g.im, fr * g.im + fi * g.re);
#pragma unroll
                for (int rr = 0; rr < RC; ++rr) {
                    const cx<float> *qr = rec[j][rr];
                    const cx<float> wx = dy * qr[2] - dz * qr[1] - dx * qr[6];
                    const cx<float> wy = dz * qr[0] - dx * qr[2] - dy * qr[6];
                    const cx<float> wz = dx * qr[1] - dy * qr[0] - dz * qr[6];
                    acc[rr][0] += f * wx + g * qr[3];
                    acc[rr][1] += f * wy + g * qr[4];
                    acc[rr][2] += f * wz + g * qr[5];
                }
            }
        }
        // sum the source slices, one right-hand side at a time
#pragma unroll
        for (int rr = 0; rr < RC; ++rr) {
            __syncthreads();
            for (int c = 0; c < 3; ++c) red[threadIdx.x][c] = acc[rr][c];
            __syncthreads();
            if (threadIdx.x < ntc && rr < rcn) {
                cx<float> s[3] = {mk(0.f, 0.f), mk(0.f, 0.f), mk(0.f, 0.f)};
                for (int q = 0; q < S; ++q)
                    for (int c = 0; c < 3; ++c) s[c] += red[q * ntc + threadIdx.x][c];
                cx<float> *o = ys + ((int64_t)(r0 + rr) * n + t0 + tc0 + threadIdx.x) * 3;
                for (int c = 0; c < 3; ++c) o[c] += s[c];
            }
        }
    }
}

// local-only lossy plans: pairs beyond the cutoff radius are skipped by a branch
template <int RC>
constexpr auto k_p2p32_cut = k_p2p32<true, RC, true>;

// The near fields of the two plans of one BEM application at once, when the interior
// plan is local only (same nodes and octree; k0 real, k1 strongly lossy; one
// right-hand side per block row): the pair geometry, the LDS staging of the source
// headers and the reciprocal square root are shared, and each pair adds k0's terms
// and, within k1's cutoff radius, k1's.  Same layout and reduction as k_p2p32.
__global__ void __launch_bounds__(TPB) k_p2p32_pair(int nleaf, int nrhs, const int32_t *__restrict__ start,
                                                    const int32_t *__restrict__ nbr,
                                                    const double *__restrict__ center,
                                                    const double *__restrict__ spts, const double *__restrict__ snrm,
                                                    const int32_t *__restrict__ stri,
                                                    const cx<float> *__restrict__ src0,
                                                    const cx<float> *__restrict__ src1, int64_t n, double k0,
                                                    double k1_re, double k1_im, float rcut2_1,
                                                    cx<float> *__restrict__ ys0, cx<float> *__restrict__ ys1) {
    constexpr int TS = 128;
    __shared__ SrcHdr32 hdr[TS];
    __shared__ __attribute__((aligned(16))) cx<float> rec[2][TS][8];   // n x a, b, n.a, unused per plan
    __shared__ int32_t sid[TS];
    __shared__ int32_t nb_start[28], nb_box[27];
    __shared__ int n_nb;
    __shared__ cx<float> red[TPB][3];
    const int box = blockIdx.x, r = blockIdx.y;
    if (box >= nleaf || r >= nrhs) return;
    const int t0 = start[box], t1 = start[box + 1];
    const int nt = t1 - t0;
    const double c0x = center[3 * box], c0y = center[3 * box + 1], c0z = center[3 * box + 2];
    if (threadIdx.x == 0) {
        int c = 0, tot = 0;
        for (int q = 0; q < 27; ++q) {
            const int b = nbr[box * 27 + q];
            if (b >= 0) {
                nb_box[c] = b;
                nb_start[c] = tot;
                tot += start[b + 1] - start[b];
                ++c;
            }
        }
        nb_start[c] = tot;
        n_nb = c;
    }
    __syncthreads();
    const int ns_total = nb_start[n_nb];
    const float krev0 = (float)(k0 * 0.15915494309189533577), kr0 = (float)k0;
    const float krev1 = (float)(k1_re * 0.15915494309189533577);
    const float kexp1 = (float)(-k1_im * 1.44269504088896340736);
    const float kr1 = (float)k1_re, ki1 = (float)k1_im;
    const float inv4pi = 0.07957747154594766788f;
    for (int tc0 = 0; tc0 < nt; tc0 += TPB) {
        const int ntc = min(TPB, nt - tc0);
        const int S = TPB / ntc;
        const int ti = threadIdx.x % ntc, sl = threadIdx.x / ntc;
        const bool active = sl < S;
        const int64_t ig = t0 + tc0 + ti;
        float tx = 0.f, ty = 0.f, tz = 0.f;
        int32_t ttri = -1;
        if (active) {
            tx = (float)(spts[3 * ig] - c0x);
            ty = (float)(spts[3 * ig + 1] - c0y);
            tz = (float)(spts[3 * ig + 2] - c0z);
            ttri = stri[ig];
        }
        cx<float> acc0[3] = {mk(0.f, 0.f), mk(0.f, 0.f), mk(0.f, 0.f)};
        cx<float> acc1[3] = {mk(0.f, 0.f), mk(0.f, 0.f), mk(0.f, 0.f)};
        for (int base = 0; base < ns_total; base += TS) {
            const int cnt = min(TS, ns_total - base);
            __syncthreads();
            for (int j = threadIdx.x; j < cnt; j += blockDim.x) {
                const int u = base + j;
                int b = 0;
                while (nb_start[b + 1] <= u) ++b;
                const int64_t sidx = start[nb_box[b]] + (u - nb_start[b]);
                SrcHdr32 q;
                q.x = (float)(spts[3 * sidx] - c0x);
                q.y = (float)(spts[3 * sidx + 1] - c0y);
                q.z = (float)(spts[3 * sidx + 2] - c0z);
                q.tri = stri[sidx];
                q.nx = (float)snrm[3 * sidx];
                q.ny = (float)snrm[3 * sidx + 1];
                q.nz = (float)snrm[3 * sidx + 2];
                q.pad = 0.f;
                hdr[j] = q;
                sid[j] = (int32_t)sidx;
            }
            __syncthreads();
            for (int e = threadIdx.x; e < cnt * 8; e += blockDim.x) {
                const int pl = (e / 4) % 2, j = e / 8;
                stage_rec32(hdr[j], (pl ? src1 : src0) + ((int64_t)r * n + sid[j]) * 7, e % 4, rec[pl][j]);
            }
            __syncthreads();
            if (!active) continue;
            for (int j = sl; j < cnt; j += S) {
                const SrcHdr32 &q = hdr[j];
                const bool self = q.tri == ttri;
                const float dx = q.x - tx, dy = q.y - ty, dz = q.z - tz;
                const float R2r = dx * dx + dy * dy + dz * dz;
                const float R2 = self ? 1.f : R2r;
                const float iR = __builtin_amdgcn_rsqf(R2);
                const float R = R2 * iR;
                const float iR2 = iR * iR;
                {
                    // k0 (real): g = e^{i k0 R} / (4 pi R), f = (i k0 R - 1) g / R^2
                    const float sn = __builtin_amdgcn_sinf(krev0 * R), cs = __builtin_amdgcn_cosf(krev0 * R);
                    const float sc = self ? 0.f : inv4pi * iR;
                    const cx<float> g = mk(sc * cs, sc * sn);
                    const float fi = kr0 * iR;
                    const cx<float> f = mk(-iR2 * g.re - fi * g.im, -iR2 * g.im + fi * g.re);
                    const cx<float> *qr = rec[0][j];
                    const cx<float> wx = dy * qr[2] - dz * qr[1] - dx * qr[6];
                    const cx<float> wy = dz * qr[0] - dx * qr[2] - dy * qr[6];
                    const cx<float> wz = dx * qr[1] - dy * qr[0] - dz * qr[6];
                    acc0[0] += f * wx + g * qr[3];
                    acc0[1] += f * wy + g * qr[4];
                    acc0[2] += f * wz + g * qr[5];
                }
                if (R2r <= rcut2_1) {
                    // k1 (lossy): the same with the decay e^{-Im k1 R}
                    const float sn = __builtin_amdgcn_sinf(krev1 * R), cs = __builtin_amdgcn_cosf(krev1 * R);
                    const float ex = __builtin_amdgcn_exp2f(kexp1 * R);
                    const float sc = self ? 0.f : inv4pi * iR * ex;
                    const cx<float> g = mk(sc * cs, sc * sn);
                    const float fr = iR2 * (-ki1 * R - 1.f), fi = kr1 * iR;
                    const cx<float> f = mk(fr * g.re - fi * g.im, fr * g.im + fi * g.re);
                    const cx<float> *qr = rec[1][j];
                    const cx<float> wx = dy * qr[2] - dz * qr[1] - dx * qr[6];
                    const cx<float> wy = dz * qr[0] - dx * qr[2] - dy * qr[6];
                    const cx<float> wz = dx * qr[1] - dy * qr[0] - dz * qr[6];
                    acc1[0] += f * wx + g * qr[3];
                    acc1[1] += f * wy + g * qr[4];
                    acc1[2] += f * wz + g * qr[5];
                }
            }
        }
        // sum the source slices, one plan at a time
        for (int pl = 0; pl < 2; ++pl) {
            __syncthreads();
            for (int c = 0; c < 3; ++c) red[threadIdx.x][c] = pl ? acc1[c] : acc0[c];
            __syncthreads();
            if (threadIdx.x < ntc) {
                cx<float> sm[3] = {mk(0.f, 0.f), mk(0.f, 0.f), mk(0.f, 0.f)};
                for (int q = 0; q < S; ++q)
                    for (int c = 0; c < 3; ++c) sm[c] += red[q * ntc + threadIdx.x][c];
                cx<float> *o = (pl ? ys1 : ys0) + ((int64_t)r * n + t0 + tc0 + threadIdx.x) * 3;
                for (int c = 0; c < 3; ++c) o[c] += sm[c];
            }
        }
    }
}

template <typename T>
__global__ void k_zero(cx<T> *__restrict__ x, int64_t m) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < m) x[i] = mk(T(0), T(0));
}

// ---------------------------------------------------------------- translations
// Batched GEMM grouped by operator: for every entry e of a tile,
//   Y[dst(e)] = T_op * X[src(e)]
// with X, Y column blocks of 3*nrhs columns of P2 complex coefficients.  The
// complex product is done as a real one: a complex column is read as its
// 2*P2 interleaved (re, im) reals and the operator is stored as the real
// 2P2 x 2P2 matrix with 2x2 blocks [[re, -im], [im, re]].
struct Tile {
    int32_t op, first, count;
};
constexpr int OS_MAXCOLS = 288;                 // columns per operator-stationary job

// Operator-stationary kernel for operators with 2 p^2 <= 98 (p <= 7; FP64 p <= 4):
// a block owns one operator and a long run of that operator's columns.  Each
// of its four waves loads the MFMA A-fragments of its RTW row tiles for the
// whole K extent into registers once (a[i][kk] = T[16 i + l%16][4 kk + l/16]),
// then the block streams the columns 16 at a time through double-buffered LDS.
// Operator traffic drops from one read per 64 columns to one read per job.
constexpr int OS_COLS = 16;

template <typename T, int KS, int RTW>
__global__ void __launch_bounds__(TPB) k_translate_os(const Tile *__restrict__ tiles, int ntiles,
                                                      const int32_t *__restrict__ ent,
                                                      const int32_t *__restrict__ src_map,
                                                      const T *__restrict__ ops, const T *__restrict__ X,
                                                      T *__restrict__ Y, int KR, int ncol, int64_t blkR, int accum) {
    constexpr int KP = KS * 4;                     // K padded to whole MFMA k-steps
    constexpr int LD = (KP * OS_COLS + TPB - 1) / TPB;
    typedef typename Mma16<T>::v4 v4;
    __shared__ T Bs[2][KP][OS_COLS];
    __shared__ int64_t s_in[OS_MAXCOLS], s_out[OS_MAXCOLS];
    const int tix = xcd_tile(blockIdx.x, ntiles);
    if (tix >= ntiles) return;
    const Tile tl = tiles[tix];
    const int C = tl.count * ncol;                 // <= OS_MAXCOLS (plan-time tiling)
    for (int c = threadIdx.x; c < C; c += blockDim.x) {
        const int e = c / ncol, cc = c % ncol;
        const int32_t en = ent[tl.first + e];
        const int32_t sb = src_map ? src_map[en] : en;
        s_in[c] = (int64_t)sb * blkR + (int64_t)cc * KR;
        s_out[c] = (int64_t)en * blkR + (int64_t)cc * KR;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const T *Top = ops + (size_t)tl.op * KR * KR;
    T a[RTW][KS];
#pragma unroll
    for (int i = 0; i < RTW; ++i) {
        const int row = (wave * RTW + i) * 16 + (lane & 15);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const int k = 4 * kk + (lane >> 4);
            a[i][kk] = (row < KR && k < KR) ? Top[(size_t)row * KR + k] : T(0);
        }
    }
    __syncthreads();
    const int ntc = (C + OS_COLS - 1) / OS_COLS;
    T pre[LD];
    auto fetch = [&](int t) {
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const int e = threadIdx.x + j * TPB;
            const int c = e / KP, k = e % KP;
            const int cg = t * OS_COLS + c;
            pre[j] = (e < KP * OS_COLS && cg < C && k < KR) ? X[s_in[cg] + k] : T(0);
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const int e = threadIdx.x + j * TPB;
            if (e < KP * OS_COLS) Bs[buf][e % KP][e / KP] = pre[j];
        }
    };
    fetch(0);
    stash(0);
    __syncthreads();
    for (int t = 0; t < ntc; ++t) {
        const int buf = t & 1;
        if (t + 1 < ntc) fetch(t + 1);
        v4 acc[RTW];
#pragma unroll
        for (int i = 0; i < RTW; ++i) acc[i] = v4{0, 0, 0, 0};
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const T b = Bs[buf][4 * kk + (lane >> 4)][lane & 15];
#pragma unroll
            for (int i = 0; i < RTW; ++i) acc[i] = Mma16<T>::mma(a[i][kk], b, acc[i]);
        }
        const int cg = t * OS_COLS + (lane & 15);
        if (cg < C) {
            T *yo = Y + s_out[cg];
#pragma unroll
            for (int i = 0; i < RTW; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = (wave * RTW + i) * 16 + Mma16<T>::row(lane >> 4, q);
                    if (row < KR) yo[row] = accum ? yo[row] + acc[i][q] : acc[i][q];
                }
        }
        if (t + 1 < ntc) stash(buf ^ 1);
        __syncthreads();
    }
}

// columns per split-BF16 job (the instantiations in launch_translate)
inline int bf3_job_cols(int p) { return p <= 5 ? 96 : (p <= 8 ? 64 : 32); }

// (of dense plans)
inline bool use_bf3(const Plan &P) {
    return P.precision == FMB_FP32 && P.translate_mode == FMB_TRANSLATE_BF16X3 && P.order >= 2;
}

// right-hand sides per translation launch: a job holds whole entries of 3 x (this many)
// columns, so wider batches run as several launches over slices of the right-hand sides
inline int translate_rhs_chunk(const Plan &P) {
    return std::min(P.nrhs_max, (use_bf3(P) ? bf3_job_cols(P.order) : OS_MAXCOLS) / 3);
}

// Split-BF16 variant of the operator-stationary kernel (FP32 plans, p <= 9).
// x = hi + lo with hi = bf16(x), lo = bf16(x - hi); a product is taken as
// a_hi b_hi + a_hi b_lo + a_lo b_hi on the 16x16x32 BF16 MFMA with FP32
// accumulation (the lo*lo term, ~2^-16 relative, is dropped).  Operators are
// pre-split at plan time and stored fragment-major: lane l of row tile i and
// k-step s holds T[16 i + l%16][32 s + 8 (l/16) + j], j = 0..7.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A job holds at most JC columns (bf3_job_cols); all of them are staged into
// LDS with one batch of loads before any MFMA runs, so a job waits for memory
// once instead of once per 16-column chunk.
// ROLE only names the launch in kernel traces: 0 S|S (M2M), 1 S|R (M2L), 2 R|R (L2L).
template <int KS, int RTW, int JC, int ROLE>
__global__ void __launch_bounds__(TPB) k_translate_bf3(const Tile *__restrict__ tiles, int ntiles,
                                                       const int32_t *__restrict__ ent,
                                                       const int32_t *__restrict__ src_map,
                                                       const bf16x8 *__restrict__ fhi,
                                                       const bf16x8 *__restrict__ flo, const float *__restrict__ X,
                                                       float *__restrict__ Y, int KR, int RT, int ncol,
                                                       int64_t blkR, int accum) {
    constexpr int KP = KS * 32;
    constexpr int CS = KP + 4;                                   // LDS column stride (floats)
    constexpr int LD = (KP * JC + TPB - 1) / TPB;
    typedef Mma16<float>::v4 v4;
    constexpr int RP = 64 * RTW + 1;                             // output tile pitch (rows of 4 waves)
    __shared__ __attribute__((aligned(16))) float Bs[JC][CS];
    __shared__ float Os[16][RP];
    __shared__ int64_t s_in[JC], s_out[JC];
    const int tix = xcd_tile(blockIdx.x, ntiles);
    if (tix >= ntiles) return;
    const Tile tl = tiles[tix];
    const int C = tl.count * ncol;                               // <= JC (plan-time tiling)
    for (int c = threadIdx.x; c < C; c += blockDim.x) {
        const int e = c / ncol, cc = c % ncol;
        const int32_t en = ent[tl.first + e];
        const int32_t sb = src_map ? src_map[en] : en;
        s_in[c] = (int64_t)sb * blkR + (int64_t)cc * KR;
        s_out[c] = (int64_t)en * blkR + (int64_t)cc * KR;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bf16x8 ah[RTW][KS], al[RTW][KS];
#pragma unroll
    for (int i = 0; i < RTW; ++i) {
        const int tile = wave * RTW + i;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (tile < RT) {
                const size_t f = (((size_t)tl.op * RT + tile) * KS + s) * 64 + lane;
                ah[i][s] = fhi[f];
                al[i][s] = flo[f];
            } else {
                for (int j = 0; j < 8; ++j) {
                    ah[i][s][j] = (__bf16)0.f;
                    al[i][s][j] = (__bf16)0.f;
                }
            }
        }
    }
    __syncthreads();
    {
        float pre[LD];
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const int e = threadIdx.x + j * TPB;
            const int c = e / KP, k = e % KP;
            pre[j] = (e < KP * JC && c < C && k < KR) ? X[s_in[c] + k] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const int e = threadIdx.x + j * TPB;
            if (e < KP * JC) Bs[e / KP][e % KP] = pre[j];
        }
    }
    __syncthreads();
    const int ntc = (C + 15) / 16;
    for (int t = 0; t < ntc; ++t) {
        v4 acc[RTW];
#pragma unroll
        for (int i = 0; i < RTW; ++i) acc[i] = v4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const float *bp = &Bs[16 * t + (lane & 15)][32 * s + 8 * (lane >> 4)];
            const float4 v0 = *reinterpret_cast<const float4 *>(bp);
            const float4 v1 = *reinterpret_cast<const float4 *>(bp + 4);
            const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            bf16x8 bh, bl;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const __bf16 h = (__bf16)v[j];
                bh[j] = h;
                bl[j] = (__bf16)(v[j] - (float)h);
            }
#pragma unroll
            for (int i = 0; i < RTW; ++i) {
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i][s], bh, acc[i], 0, 0, 0);
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i][s], bl, acc[i], 0, 0, 0);
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i][s], bh, acc[i], 0, 0, 0);
            }
        }
        // the 16 x KR output tile goes through LDS so that every column is
        // written as one contiguous run of KR floats
#pragma unroll
        for (int i = 0; i < RTW; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) Os[lane & 15][(wave * RTW + i) * 16 + 4 * (lane >> 4) + q] = acc[i][q];
        __syncthreads();
        const int cn = min(16, C - 16 * t);
        for (int e = threadIdx.x; e < cn * KR; e += TPB) {
            const int c = e / KR, row = e % KR;
            float *yo = Y + s_out[16 * t + c] + row;
            *yo = accum ? *yo + Os[c][row] : Os[c][row];
        }
        __syncthreads();
    }
}

// plan-time split of FP32 operators into fragment-major BF16 hi/lo parts
__global__ void k_split_bf16(const float *__restrict__ T, int nops, int KR, int RT, int KS, bf16x8 *__restrict__ hi,
                             bf16x8 *__restrict__ lo) {
    const int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)nops * RT * KS * 64;
    if (f >= total) return;
    const int lane = (int)(f % 64);
    const int s = (int)((f / 64) % KS);
    const int tile = (int)((f / (64 * KS)) % RT);
    const int64_t op = f / ((int64_t)64 * KS * RT);
    const int row = 16 * tile + (lane & 15);
    bf16x8 h, l;
    for (int j = 0; j < 8; ++j) {
        const int k = 32 * s + 8 * (lane >> 4) + j;
        const float x = (row < KR && k < KR) ? T[((size_t)op * KR + row) * KR + k] : 0.f;
        const __bf16 xh = (__bf16)x;
        h[j] = xh;
        l[j] = (__bf16)(x - (float)xh);
    }
    hi[f] = h;
    lo[f] = l;
}

template <int ROLE>
void launch_bf3(int p, unsigned g, const Tile *tiles, int64_t ntiles, const int32_t *ent, const int32_t *src_map,
                const bf16x8 *h, const bf16x8 *l, const float *x, float *y, int KR, int RT, int ncol, int64_t blkR,
                int accum, hipStream_t s) {
    const int nt = (int)ntiles;
    switch (p) {
        case 2:
        case 3:
        case 4: k_translate_bf3<1, 1, 96, ROLE><<<g, TPB, 0, s>>>(tiles, nt, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum); break;
        case 5: k_translate_bf3<2, 1, 96, ROLE><<<g, TPB, 0, s>>>(tiles, nt, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum); break;
        case 6: k_translate_bf3<3, 2, 64, ROLE><<<g, TPB, 0, s>>>(tiles, nt, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum); break;
        case 7:
        case 8: k_translate_bf3<4, 2, 64, ROLE><<<g, TPB, 0, s>>>(tiles, nt, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum); break;
        default: k_translate_bf3<6, 3, 32, ROLE><<<g, TPB, 0, s>>>(tiles, nt, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum); break;
    }
}

// role: 0 S|S, 1 S|R, 2 R|R (names the split-BF16 launches in kernel traces);
// accum: add the products into Y instead of overwriting it
template <typename T>
void launch_translate(const Tile *tiles, int64_t ntiles, const int32_t *ent, const int32_t *src_map, const T *ops,
                      const T *x, T *y, int KR, int ncol, int64_t blkR, hipStream_t s, int role, int accum,
                      const void *fhi, const void *flo) {
    if (ntiles <= 0) return;
    const int p = (int)lround(sqrt(KR / 2.0));
    const unsigned g = (unsigned)(((ntiles + 7) / 8) * 8);
    if constexpr (sizeof(T) == sizeof(float)) {
        if (fhi) {
            // split-BF16 translations (checked by use_bf3)
            const int RT = (KR + 15) / 16;
            // register tiles per instantiation below: KS k-steps of 32, 4 waves x RTW row tiles of 16
            static const int ks_of[10] = {0, 0, 1, 1, 1, 2, 3, 4, 4, 6}, rtw_of[10] = {0, 0, 1, 1, 1, 1, 2, 2, 2, 3};
            if (p < 2 || p > 9 || 2 * p * p != KR || (KR + 31) / 32 != ks_of[p] || RT > 4 * rtw_of[p])
                throw std::runtime_error("split-BF16 translation: unsupported operator size");
            const bf16x8 *h = (const bf16x8 *)fhi, *l = (const bf16x8 *)flo;
            switch (role) {
                case 0: launch_bf3<0>(p, g, tiles, ntiles, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum, s); break;
                case 1: launch_bf3<1>(p, g, tiles, ntiles, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum, s); break;
                default: launch_bf3<2>(p, g, tiles, ntiles, ent, src_map, h, l, x, y, KR, RT, ncol, blkR, accum, s); break;
            }
            FMB_LAUNCH_CHECK();
            return;
        }
    }
    auto go = [&](auto kern) { kern<<<g, TPB, 0, s>>>(tiles, (int)ntiles, ent, src_map, ops, x, y, KR, ncol, blkR, accum); };
    if constexpr (sizeof(T) == sizeof(float)) {
        switch (p) {
            case 1: go(k_translate_os<T, 1, 1>); break;
            case 2: go(k_translate_os<T, 2, 1>); break;
            case 3: go(k_translate_os<T, 5, 1>); break;
            case 4: go(k_translate_os<T, 8, 1>); break;
            case 5: go(k_translate_os<T, 13, 1>); break;
            case 6: go(k_translate_os<T, 18, 2>); break;
            case 7: go(k_translate_os<T, 25, 2>); break;
            default: throw std::runtime_error("FP32 translation: unsupported operator size");
        }
    } else {
        switch (p) {
            case 1: go(k_translate_os<T, 1, 1>); break;
            case 2: go(k_translate_os<T, 2, 1>); break;
            case 3: go(k_translate_os<T, 5, 1>); break;
            case 4: go(k_translate_os<T, 8, 1>); break;
            default: throw std::runtime_error("FP64 translation: unsupported operator size");
        }
    }
    FMB_LAUNCH_CHECK();
}

// parent (level l) multipole = sum of its children's translated slots
// Column sums of a row range [e0, e1) of slots (rows of blk complex values, the
// first ncolP2 of which are used) by one block: columns go in chunks of
// CW = min(ncolP2, 128) (FP64: 32, so that a column's sum does not depend on the
// number of right-hand sides); within a chunk G = TPB / CW row groups take rows
// e0 + g, e0 + g + G, ... and their partial sums are added in group order, so
// the result does not depend on timing.
template <typename T>
__device__ inline void slot_sum(const cx<T> *__restrict__ Y, int e0, int e1, int64_t blk, int ncolP2,
                                cx<T> *__restrict__ out, bool accumulate, cx<T> *sm) {
    const int t = threadIdx.x;
    const int CW = sizeof(T) == 8 ? 32 : min(ncolP2, 128), G = TPB / CW;
    const int g = t / CW, c = t % CW;
    for (int c0 = 0; c0 < ncolP2; c0 += CW) {
        const int cw = min(CW, ncolP2 - c0);
        cx<T> s = mk(T(0), T(0));
        if (g < G && c < cw) {
#pragma unroll 4
            for (int e = e0 + g; e < e1; e += G) s += Y[(int64_t)e * blk + c0 + c];
        }
        sm[t] = s;
        __syncthreads();
        if (t < cw) {
            cx<T> tot = sm[t];
            for (int q = 1; q < G; ++q) tot += sm[q * CW + t];
            if (accumulate) out[c0 + t] += tot;
            else out[c0 + t] = tot;
        }
        __syncthreads();
    }
}

// parent multipole = sum of its children's S|S slots
template <typename T>
__global__ void __launch_bounds__(TPB) k_sum_children(const int32_t *__restrict__ child_start, int64_t nbox,
                                                      const cx<T> *__restrict__ Yc, cx<T> *__restrict__ Mp, int64_t blk,
                                                      int ncolP2) {
    __shared__ cx<T> sm[TPB];
    const int64_t b = blockIdx.x;
    slot_sum(Yc, child_start[b], child_start[b + 1], blk, ncolP2, Mp + b * blk, false, sm);
}

// The S|R slot sums of every level in one launch: block b belongs to the level
// l with box0[l] <= b < box0[l + 1]; that level's box b - box0[l] sums its
// slots into its local expansion (overwriting it).
struct FarSumLevels {
    int nlev;
    int64_t box0[MAX_DEPTH + 2];
    const int32_t *ff_ofs[MAX_DEPTH + 1];
    int64_t slot_base[MAX_DEPTH + 1];
    void *L[MAX_DEPTH + 1];
};

template <typename T>
__global__ void __launch_bounds__(TPB) k_sum_far_all(FarSumLevels lv, const cx<T> *__restrict__ Yf, int64_t blk,
                                                     int ncolP2) {
    __shared__ cx<T> sm[TPB];
    const int64_t gb = blockIdx.x;
    int l = 0;
    while (l + 1 < lv.nlev && lv.box0[l + 1] <= gb) ++l;
    const int64_t b = gb - lv.box0[l];
    const int32_t *ofs = lv.ff_ofs[l];
    slot_sum(Yf + lv.slot_base[l] * blk, ofs[b], ofs[b + 1], blk, ncolP2, (cx<T> *)lv.L[l] + b * blk, false, sm);
}

inline unsigned gridn(int64_t m, int tpb = TPB) { return (unsigned)((m + tpb - 1) / tpb); }

// One product is a fixed sequence of steps (a launch or a short run of
// launches); matvec_step issues step number `step` and returns false past the
// last one, so that two products on two streams can be issued alternately.
template <typename T>
bool matvec_step(Plan &P, const cx<T> *a, const cx<T> *b, cx<T> *y, int nrhs, hipStream_t s, int step) {
    const int64_t n = P.n;
    const int L = P.depth, p = P.order, P2 = P.P2;
    const int64_t blk = (int64_t)P.nrhs_max * 3 * P2;
    const int ncol = 3 * nrhs;
    const int KR = 2 * P2;                          // real rows of the embedded operators
    const int64_t blkR = 2 * blk;
    const bool bf3 = use_bf3(P);
    // translations run over slices of at most cw right-hand sides; roff(r0) is the
    // offset (in reals) of right-hand side r0 inside a box's or slot's block
    const int cw = translate_rhs_chunk(P);
    auto roff = [&](int r0) { return (int64_t)r0 * 3 * KR; };
    cx<T> *src = P.src.as<cx<T>>();
    cx<T> *ys = P.ys.as<cx<T>>();
    cx<T> *yb = P.ybuf.as<cx<T>>();
    StageTimer &tm = P.timer;
    hipEvent_t ev = nullptr;
    int k = 0;
    if (step == k++) {
        tm.begin(ST_GATHER, s, ev);
        k_gather_src<T><<<gridn(n), TPB, 0, s>>>(a, b, P.perm.as<int32_t>(), P.sw.as<double>(), P.snrm.as<double>(), n,
                                                 nrhs, src);
        FMB_LAUNCH_CHECK();
        tm.end(ST_GATHER, s, ev);
        return true;
    }
    // Step 1: leaf multipoles
    Level &LL = P.lv[L];
    const bool far = P.far_on();
    const int lmin = std::max(2, P.far_lmin);
    if (step == k++) {
        if (!far) return true;
        FMB_REQUIRE(p <= 40, "leaf order too large for the multipole kernel");
        const bool wide = p2m_wide<T>(P);
        auto kern = wide ? k_p2m<T, 16> : k_p2m<T, 8>;
        const size_t sh = wide ? p2m_lds<T, 16>(p) : p2m_lds<T, 8>(p);
        leaf_lds_limit(kern, sh);
        tm.begin(ST_P2M, s, ev);
        kern<<<dim3((unsigned)LL.nbox, (unsigned)nrhs), 64 * (p / 8 + 1), sh, s>>>(
            LL.start.as<int32_t>(), P.lnode.as<LeafNode<T>>(), P.snrm.as<double>(), src, n, p, P.k_re, P.k_im,
            P.inv_alpha.as<double>() + (size_t)L * p, P.btab.as<T>(), P.nrhs_max, LL.M.as<cx<T>>());
        FMB_LAUNCH_CHECK();
        tm.end(ST_P2M, s, ev);
        return true;
    }
    // Step 2: upward pass (S|S), levels L-1 .. 2
    for (int l = L - 1; l >= 2; --l) {
        Level &V = P.lv[l], &C = P.lv[l + 1];
        if (step != k++) continue;
        if (l < lmin) return true;
        if (!P.dense) {
            tm.begin(ST_M2M, s, ev);
            tm.end(ST_M2M, s, ev, hf_m2m<T>(P, l, nrhs, s));
            return true;
        }
        if (V.ntiles_m2m == 0) return true;
        tm.begin(ST_M2M, s, ev);
        for (int r0 = 0; r0 < nrhs; r0 += cw)
            launch_translate<T>(V.tiles_m2m.as<Tile>(), V.ntiles_m2m, C.by_octant.as<int32_t>(), nullptr, V.m2m.as<T>(),
                                (const T *)C.M.p + roff(r0), (T *)yb + roff(r0), KR, 3 * std::min(cw, nrhs - r0),
                                blkR, s, 0, 0, bf3 ? V.m2m_hi.p : nullptr, V.m2m_lo.p);
        tm.end(ST_M2M, s, ev, (nrhs + cw - 1) / cw);
        tm.begin(ST_SUMS, s, ev);
        k_sum_children<T><<<(unsigned)V.nbox, TPB, 0, s>>>(V.child_start.as<int32_t>(), V.nbox, yb, V.M.as<cx<T>>(), blk,
                                                           ncol * P2);
        FMB_LAUNCH_CHECK();
        tm.end(ST_SUMS, s, ev);
        return true;
    }
    // Step 3a: S|R of every level, one run of launches; each level's slots have
    // their own region of the slot buffer (slot_base)
    if (step == k++) {
        if (!far) return true;
        int nk = 0;
        tm.begin(ST_M2L, s, ev);
        if (!P.dense) {
            // each target sums its own far-field translations and writes its local expansion; the finest
            // level has a launch of its own while its timer is on
            const bool split = tm.mask >> ST_M2L_FINE & 1u;
            nk = hf_m2l<T>(P, lmin, split ? L - 1 : L, nrhs, s);
            if (split) {
                hipEvent_t ev2 = nullptr;
                tm.begin(ST_M2L_FINE, s, ev2);
                const int fine = hf_m2l<T>(P, L, L, nrhs, s);
                tm.end(ST_M2L_FINE, s, ev2, fine);
                nk += fine;
            }
            tm.end(ST_M2L, s, ev, nk);
            return true;
        }
        for (int l = lmin; l <= L; ++l) {
            Level &V = P.lv[l];
            if (V.ntiles_m2l == 0) continue;
            for (int r0 = 0; r0 < nrhs; r0 += cw) {
                launch_translate<T>(V.tiles_m2l.as<Tile>(), V.ntiles_m2l, V.ff_by_op.as<int32_t>(),
                                    V.ff_src.as<int32_t>(), V.m2l.as<T>(), (const T *)V.M.p + roff(r0),
                                    (T *)(yb + V.slot_base * blk) + roff(r0), KR, 3 * std::min(cw, nrhs - r0), blkR,
                                    s, 1, 0, bf3 ? V.m2l_hi.p : nullptr, V.m2l_lo.p);
                ++nk;
            }
        }
        tm.end(ST_M2L, s, ev, nk);
        return true;
    }
    // Step 3b: the S|R slot sums of every level (one launch, overwriting L),
    // then R|R from the parent added into each level in turn
    if (step == k++) {
        if (!far || !P.dense) return true;
        FarSumLevels fs{};
        fs.nlev = L - lmin + 1;
        int64_t tot = 0;
        for (int l = lmin; l <= L; ++l) {
            Level &V = P.lv[l];
            fs.box0[l - lmin] = tot;
            fs.ff_ofs[l - lmin] = V.ff_ofs.as<int32_t>();
            fs.slot_base[l - lmin] = V.slot_base;
            fs.L[l - lmin] = V.L.p;
            tot += V.nbox;
        }
        fs.box0[L - lmin + 1] = tot;
        tm.begin(ST_SUMS, s, ev);
        k_sum_far_all<T><<<(unsigned)tot, TPB, 0, s>>>(fs, yb, blk, ncol * P2);
        FMB_LAUNCH_CHECK();
        tm.end(ST_SUMS, s, ev);
        return true;
    }
    for (int l = 3; l <= L; ++l) {
        Level &V = P.lv[l];
        if (step != k++) continue;
        if (l <= lmin) return true;
        if (!P.dense) {
            tm.begin(ST_L2L, s, ev);
            tm.end(ST_L2L, s, ev, hf_l2l<T>(P, l, nrhs, s));
            return true;
        }
        if (V.ntiles_l2l == 0) return true;
        Level &U = P.lv[l - 1];
        tm.begin(ST_L2L, s, ev);
        for (int r0 = 0; r0 < nrhs; r0 += cw)
            launch_translate<T>(V.tiles_l2l.as<Tile>(), V.ntiles_l2l, V.by_octant.as<int32_t>(), V.parent.as<int32_t>(),
                                V.l2l.as<T>(), (const T *)U.L.p + roff(r0), (T *)V.L.p + roff(r0), KR,
                                3 * std::min(cw, nrhs - r0), blkR, s, 2, 1, bf3 ? V.l2l_hi.p : nullptr, V.l2l_lo.p);
        tm.end(ST_L2L, s, ev, (nrhs + cw - 1) / cw);
        return true;
    }
    // Step 4: local expansions at the targets, then the near sum
    if (step == k++) {
        if (!far) {
            // local-only plan: the near sum accumulates onto zero
            k_zero<T><<<gridn((int64_t)nrhs * n * 3), TPB, 0, s>>>(ys, (int64_t)nrhs * n * 3);
            FMB_LAUNCH_CHECK();
            return true;
        }
        tm.begin(ST_L2P, s, ev);
        launch_l2p<T>(P, nrhs, LL.L.as<cx<T>>(), ys, s);
        tm.end(ST_L2P, s, ev);
        return true;
    }
    if (step == k++) {
        if (P.fuse_p2p) return true;           // the two-product runner launches both near fields at once
        tm.begin(ST_P2P, s, ev);
        if (sizeof(T) == sizeof(float)) {
            const bool lossy = P.k_im != 0.0;
            const int rc = nrhs >= 8 ? 8 : (nrhs >= 4 ? 4 : (nrhs >= 2 ? 2 : 1));
            decltype(&k_p2p32<true, 1>) kern;
            switch (rc) {
                case 8: kern = lossy ? k_p2p32<true, 8> : k_p2p32<false, 8>; break;
                case 4: kern = lossy ? k_p2p32<true, 4> : k_p2p32<false, 4>; break;
                case 2: kern = lossy ? k_p2p32<true, 2> : k_p2p32<false, 2>; break;
                default: kern = lossy ? k_p2p32<true, 1> : k_p2p32<false, 1>; break;
            }
            if (!far) {
                switch (rc) {
                    case 8: kern = k_p2p32_cut<8>; break;
                    case 4: kern = k_p2p32_cut<4>; break;
                    case 2: kern = k_p2p32_cut<2>; break;
                    default: kern = k_p2p32_cut<1>; break;
                }
            }
            kern<<<dim3((unsigned)LL.nbox, (unsigned)((nrhs + rc - 1) / rc)), TPB, 0, s>>>(
                (int)LL.nbox, nrhs, LL.start.as<int32_t>(), LL.nbr.as<int32_t>(), LL.center.as<double>(),
                P.spts.as<double>(), P.snrm.as<double>(), P.stri.as<int32_t>(), (const cx<float> *)src, n, P.k_re,
                P.k_im, (float)std::min(P.rcut2, 1e30), (cx<float> *)ys);
        } else {
            auto kern = P.k_im != 0.0 ? k_p2p64<true> : k_p2p64<false>;
            kern<<<dim3((unsigned)LL.nbox, nrhs), TPB, 0, s>>>(
                LL.start.as<int32_t>(), LL.nbr.as<int32_t>(), P.spts.as<double>(), P.snrm.as<double>(),
                P.stri.as<int32_t>(), (const cx<double> *)src, n, P.k_re, P.k_im, P.rcut2, (cx<double> *)ys);
        }
        FMB_LAUNCH_CHECK();
        tm.end(ST_P2P, s, ev);
        return true;
    }
    if (step != k++) return false;
    if (P.corr_mode != FMB_CORR_NONE) {
        // back to user order with the self-triangle terms added in the same pass
        tm.begin(ST_CORR, s, ev);
        scatter_with_corrections(P, ys, a, b, y, nrhs, s);
        tm.end(ST_CORR, s, ev);
    } else {
        tm.begin(ST_SCATTER, s, ev);
        k_scatter_out<T><<<gridn(n), TPB, 0, s>>>(ys, P.perm.as<int32_t>(), n, nrhs, y);
        FMB_LAUNCH_CHECK();
        tm.end(ST_SCATTER, s, ev);
    }
    return true;
}

}  // namespace

// target job count per launch: about 12 resident blocks on each of the 256 CUs
constexpr int64_t EP_BLOCKS = 3072;

// Dense operators serve plans of one small order: there one small GEMM per offset costs less than walking a class's
// tiles through LDS.  FP32 up to order 7, 9 with split-BF16 products.  One product, dense against rotation / shift
// (ms; torus 60,000 nodes, sphere 3,840): FP32 p = 7 0.60 / 0.57, 0.212 / 0.227; p = 8 0.81 / 0.69, 0.29 / 0.24;
// split-BF16 p = 9 0.76 / 0.81, 0.235 / 0.263; FP32 p = 1 0.172 / 0.241, 0.054 / 0.077.  FP64 up to order 4 (p = 1
// 0.264 / 0.386, 0.059 / 0.100; p = 4 0.363 / 0.459, 0.085 / 0.115): above it the slots, which hold the result of every
// pair, outgrow what they save (GEMMs of the larger FP64 operators p = 5 0.76 / 0.49, 0.161 / 0.124; p = 9 1.85 / 0.81,
// 0.347 / 0.192 and 846 / 103 MB).
bool dense_order(int precision, int translate_mode, int p) {
    if (precision == FMB_FP64) return p <= 4;
    return p <= (translate_mode == FMB_TRANSLATE_BF16X3 ? 9 : 7);
}

void build_tiles(Plan &P, hipStream_t s) {
    const int L = P.depth;
    auto upload = [&](std::vector<Tile> &v, DevBuf &buf, int64_t &cnt) {
        cnt = (int64_t)v.size();
        buf.alloc(std::max<size_t>(1, v.size()) * sizeof(Tile));
        if (!v.empty())
            FMB_CHECK_HIP(hipMemcpyAsync(buf.p, v.data(), v.size() * sizeof(Tile), hipMemcpyHostToDevice, s));
    };
    // entries per tile.  Operator-stationary jobs hold up to OS_MAXCOLS columns;
    // shorter jobs are used until a level spreads over about EP_BLOCKS blocks:
    // a job walks its columns one 16-column chunk after another, so the level's
    // time is set by the longest chain of gathered loads, not by operator traffic.
    const int cols = use_bf3(P) ? bf3_job_cols(P.order) : OS_MAXCOLS;
    const int cw = translate_rhs_chunk(P);
    const int ep_max = std::max(1, cols / (3 * cw));
    const int ep_min = std::max(1, OS_COLS / (3 * cw));
    auto ep_for = [&](int64_t total) {
        int64_t e = total / EP_BLOCKS;
        return (int)std::max<int64_t>(ep_min, std::min<int64_t>(ep_max, e));
    };
    auto chunk = [](std::vector<Tile> &v, int ep, int op, int first, int count) {
        for (int q = 0; q < count; q += ep) v.push_back(Tile{op, first + q, std::min(ep, count - q)});
    };
    for (int l = std::max(2, P.far_lmin); l <= L; ++l) {
        Level &V = P.lv[l];
        std::vector<Tile> t;
        const int e2l = ep_for(V.nff);
        for (int o = 0; o < N_M2L_OPS; ++o) chunk(t, e2l, o, V.op_start[o], V.op_start[o + 1] - V.op_start[o]);
        upload(t, V.tiles_m2l, V.ntiles_m2l);
        if (l < L) {
            Level &C = P.lv[l + 1];
            std::vector<Tile> u;
            const int e = ep_for(C.nbox);
            for (int o = 0; o < 8; ++o) chunk(u, e, o, C.oct_start[o], C.oct_start[o + 1] - C.oct_start[o]);
            upload(u, V.tiles_m2m, V.ntiles_m2m);
        }
        if (l >= 3 && l > P.far_lmin) {
            std::vector<Tile> u;
            const int e = ep_for(V.nbox);
            for (int o = 0; o < 8; ++o) chunk(u, e, o, V.oct_start[o], V.oct_start[o + 1] - V.oct_start[o]);
            upload(u, V.tiles_l2l, V.ntiles_l2l);
        }
    }
    FMB_CHECK_HIP(hipStreamSynchronize(s));
}

void split_operators(Plan &P, hipStream_t s) {
    if (!use_bf3(P)) return;
    const int KR = 2 * P.P2, RT = (KR + 15) / 16, KS = (KR + 31) / 32;
    auto split = [&](const DevBuf &T, int nops, DevBuf &hi, DevBuf &lo) {
        if (!T.p) return;
        const int64_t total = (int64_t)nops * RT * KS * 64;
        hi.alloc(total * sizeof(bf16x8));
        lo.alloc(total * sizeof(bf16x8));
        k_split_bf16<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(T.as<float>(), nops, KR, RT, KS, hi.as<bf16x8>(),
                                                                      lo.as<bf16x8>());
        FMB_LAUNCH_CHECK();
    };
    for (int l = std::max(2, P.far_lmin); l <= P.depth; ++l) {
        Level &V = P.lv[l];
        split(V.m2l, N_M2L_OPS, V.m2l_hi, V.m2l_lo);
        if (l < P.depth) split(V.m2m, 8, V.m2m_hi, V.m2m_lo);
        if (l >= 3 && l > P.far_lmin) split(V.l2l, 8, V.l2l_hi, V.l2l_lo);
    }
    FMB_CHECK_HIP(hipStreamSynchronize(s));
}

void alloc_workspace(Plan &P) {
    const size_t esz = P.precision == FMB_FP64 ? sizeof(cx<double>) : sizeof(cx<float>);
    const int64_t blk = (int64_t)P.nrhs_max * 3 * P.P2;
    if (!P.dense) {
        // the translations need no slot buffer
        for (int l = std::max(2, P.far_lmin); l <= P.depth; ++l) {
            Level &V = P.lv[l];
            const int64_t b = (int64_t)P.nrhs_max * 3 * V.p * V.p;
            V.M.alloc((size_t)V.nbox * b * esz);
            V.L.alloc((size_t)V.nbox * b * esz);
        }
        P.ybuf.alloc(256);
        P.src.alloc((size_t)P.nrhs_max * P.n * 7 * esz);
        P.ys.alloc((size_t)P.nrhs_max * P.n * 3 * esz);
        return;
    }
    // S|R slots of all levels side by side (they are written in one run of
    // launches); the S|S slots of the upward pass reuse the front of the buffer
    int64_t slots = 1, sr = 0;
    for (int l = std::max(2, P.far_lmin); l <= P.depth; ++l) {
        Level &V = P.lv[l];
        V.M.alloc((size_t)V.nbox * blk * esz);
        V.L.alloc((size_t)V.nbox * blk * esz);
        V.slot_base = sr;
        sr += V.nff;
        if (l < P.depth) slots = std::max<int64_t>(slots, P.lv[l + 1].nbox);
    }
    slots = std::max(slots, sr);
    P.ybuf.alloc((size_t)slots * blk * esz);
    P.src.alloc((size_t)P.nrhs_max * P.n * 7 * esz);
    P.ys.alloc((size_t)P.nrhs_max * P.n * 3 * esz);
}

hipEvent_t StageTimer::get() {
    if (!pool.empty()) {
        hipEvent_t e = pool.back();
        pool.pop_back();
        return e;
    }
    hipEvent_t e;
    FMB_CHECK_HIP(hipEventCreate(&e));
    return e;
}

void StageTimer::begin(int st, hipStream_t s, hipEvent_t &e0) {
    if (!(mask >> st & 1u)) return;
    e0 = get();
    FMB_CHECK_HIP(hipEventRecord(e0, s));
}

void StageTimer::end(int st, hipStream_t s, hipEvent_t e0, int nk) {
    if (!(mask >> st & 1u)) return;
    hipEvent_t e1 = get();
    FMB_CHECK_HIP(hipEventRecord(e1, s));
    pending[st].push_back({e0, e1});
    pending_nk[st].push_back(nk);
    if (pending[st].size() > 4096) collect();
}

void StageTimer::collect() {
    for (int st = 0; st < ST_COUNT; ++st) {
        for (size_t i = 0; i < pending[st].size(); ++i) {
            auto &pr = pending[st][i];
            FMB_CHECK_HIP(hipEventSynchronize(pr.second));
            float ms_ = 0.f;
            FMB_CHECK_HIP(hipEventElapsedTime(&ms_, pr.first, pr.second));
            ms[st] += ms_;
            launches[st] += pending_nk[st][i];
            pool.push_back(pr.first);
            pool.push_back(pr.second);
        }
        pending[st].clear();
        pending_nk[st].clear();
    }
}

void StageTimer::reset() {
    collect();
    for (int st = 0; st < ST_COUNT; ++st) {
        ms[st] = 0;
        launches[st] = 0;
    }
}

StageTimer::~StageTimer() {
    for (int st = 0; st < ST_COUNT; ++st)
        for (auto &pr : pending[st]) {
            (void)hipEventDestroy(pr.first);
            (void)hipEventDestroy(pr.second);
        }
    for (hipEvent_t e : pool) (void)hipEventDestroy(e);
}

// The adjoint product shares the forward steps from P2M through the last
// R|R level (its sources are monopole charges in the forward record layout);
// gather, L2P, P2P and the return to user order are its own.
static bool adjoint_step(Plan &P, const void *y, void *abar, void *bbar, int nrhs, hipStream_t s, int step) {
    const int nmid = 3 + 2 * std::max(P.depth - 2, 0);
    StageTimer &tm = P.timer;
    hipEvent_t ev = nullptr;
    if (step == 0) {
        tm.begin(ST_GATHER, s, ev);
        adjoint_gather(P, y, nrhs, s);
        tm.end(ST_GATHER, s, ev);
        return true;
    }
    if (step <= nmid) {
        if (P.precision == FMB_FP64) return matvec_step<double>(P, nullptr, nullptr, nullptr, nrhs, s, step);
        return matvec_step<float>(P, nullptr, nullptr, nullptr, nrhs, s, step);
    }
    if (step == nmid + 1) {
        tm.begin(ST_L2P, s, ev);
        adjoint_l2p(P, nrhs, s);
        tm.end(ST_L2P, s, ev);
        return true;
    }
    if (step == nmid + 2) {
        tm.begin(ST_P2P, s, ev);
        adjoint_p2p(P, nrhs, s);
        tm.end(ST_P2P, s, ev);
        return true;
    }
    if (step == nmid + 3) {
        tm.begin(ST_CORR, s, ev);
        adjoint_finish(P, y, abar, bbar, nrhs, s);
        tm.end(ST_CORR, s, ev);
        return true;
    }
    return false;
}

static bool run_step(Plan &P, const void *a, const void *b, void *y, int nrhs, hipStream_t s, int step) {
    if (P.precision == FMB_FP64)
        return matvec_step<double>(P, (const cx<double> *)a, (const cx<double> *)b, (cx<double> *)y, nrhs, s, step);
    return matvec_step<float>(P, (const cx<float> *)a, (const cx<float> *)b, (cx<float> *)y, nrhs, s, step);
}

void run_matvec(Plan &P, const void *a, const void *b, void *y, int nrhs, hipStream_t s) {
    for (int st = 0; run_step(P, a, b, y, nrhs, s, st); ++st) {
    }
}

void run_matvec_adjoint(Plan &P, const void *y, void *abar, void *bbar, int nrhs, hipStream_t s) {
    adjoint_prepare(P);
    for (int st = 0; adjoint_step(P, y, abar, bbar, nrhs, s, st); ++st) {
    }
}

// the two plans of one BEM application share their nodes and octree when both are
// FP32 over the same points at the same depth.  When the interior plan is local only
// (its product is a cut near field and little else), both near fields run as one
// launch.  When both plans have far fields, their products overlap on two streams,
// and joining them around one near-field launch measured slower (the 60k-node torus:
// 316 against 303 ms per mixed solve), so they stay apart.
static bool p2p_fusable(const Plan &P0, const Plan &P1) {
    return P0.precision == FMB_FP32 && P1.precision == FMB_FP32 && &P0 != &P1 && P0.n == P1.n &&
           P0.depth == P1.depth && P0.lv[P0.depth].nbox == P1.lv[P1.depth].nbox && P0.k_im == 0.0 &&
           P1.k_im > 0.0 && P0.far_on() && !P1.far_on() && P0.lo[0] == P1.lo[0] && P0.lo[1] == P1.lo[1] &&
           P0.lo[2] == P1.lo[2] && P0.ext == P1.ext;
}

// two events per device and host thread for the join around the fused near field
static hipEvent_t *pair_events() {
    static thread_local std::map<int, std::array<hipEvent_t, 2>> evs;
    int dev = 0;
    FMB_CHECK_HIP(hipGetDevice(&dev));
    auto it = evs.find(dev);
    if (it == evs.end()) {
        std::array<hipEvent_t, 2> e{};
        for (auto &x : e) FMB_CHECK_HIP(hipEventCreateWithFlags(&x, hipEventDisableTiming));
        it = evs.emplace(dev, e).first;
    }
    return it->second.data();
}

static void launch_p2p_pair(Plan &P0, Plan &P1, int nrhs, hipStream_t s) {
    Level &LL = P0.lv[P0.depth];
    hipEvent_t ev = nullptr;
    P0.timer.begin(ST_P2P, s, ev);
    k_p2p32_pair<<<dim3((unsigned)LL.nbox, (unsigned)nrhs), TPB, 0, s>>>(
        (int)LL.nbox, nrhs, LL.start.as<int32_t>(), LL.nbr.as<int32_t>(), LL.center.as<double>(),
        P0.spts.as<double>(), P0.snrm.as<double>(), P0.stri.as<int32_t>(), P0.src.as<cx<float>>(),
        P1.src.as<cx<float>>(), P0.n, P0.k_re, P1.k_re, P1.k_im, (float)std::min(P1.rcut2, 1e30),
        P0.ys.as<cx<float>>(), P1.ys.as<cx<float>>());
    FMB_LAUNCH_CHECK();
    P0.timer.end(ST_P2P, s, ev);
}

void run_matvec_pair(Plan &P0, const void *a0, const void *b0, void *y0, hipStream_t s0, Plan &P1, const void *a1,
                     const void *b1, void *y1, hipStream_t s1, int nrhs) {
    // the near-field step (the same index in both plans: gather, P2M, the S|S levels, S|R, its sums,
    // the R|R levels, L2P, then P2P)
    const bool fuse = p2p_fusable(P0, P1);
    const int p2p_step = 2 * P0.depth + 1;
    P0.fuse_p2p = P1.fuse_p2p = fuse;
    struct Reset {
        Plan &a, &b;
        ~Reset() { a.fuse_p2p = b.fuse_p2p = false; }
    } reset{P0, P1};
    bool more0 = true, more1 = true;
    for (int st = 0; more0 || more1; ++st) {
        if (more0) more0 = run_step(P0, a0, b0, y0, nrhs, s0, st);
        if (more1) more1 = run_step(P1, a1, b1, y1, nrhs, s1, st);
        if (fuse && st == p2p_step) {
            // s0 waits for s1's L2P, runs both near fields, and s1 waits for that
            hipEvent_t *ev = pair_events();
            if (s0 != s1) {
                FMB_CHECK_HIP(hipEventRecord(ev[0], s1));
                FMB_CHECK_HIP(hipStreamWaitEvent(s0, ev[0], 0));
            }
            launch_p2p_pair(P0, P1, nrhs, s0);
            if (s0 != s1) {
                FMB_CHECK_HIP(hipEventRecord(ev[1], s0));
                FMB_CHECK_HIP(hipStreamWaitEvent(s1, ev[1], 0));
            }
        }
    }
}

}  // namespace fmb
