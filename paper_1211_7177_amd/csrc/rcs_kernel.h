// Translations by rotation, coaxial shift and rotation back on the matrix cores:
// the kernel, one instantiation per order.
//
// A translation by t with angles (theta, phi) of a coefficient vector c is
//   1. c'_n^m' = sum_m W^n_{m m'}(theta) e^{i m phi} c_n^m
//   2. c''_q^m = sum_n C^|m|_{q n}(|t|) c'_n^m
//   3. d_q^m'  = e^{-i m' phi} sum_m W^q_{m' m}(theta) c''_q^m
// (hf.hip derives W and C).  Three properties make it dense work of small
// matrices over many columns:
// * W^n_{-m,-m'} = W^n_{m m'}: in the combinations (x_m +- x_-m)/sqrt 2 each
//   degree splits into an (n+1) x (n+1) and an n x n orthogonal block, which
//   halves the rotations' work;
// * W^n_{m' m} = (-1)^(m+m') W^n_{m m'}: the rotation back reads the blocks of
//   the rotation forth; its signs go into C and into the closing phases;
// * a reflection in z, c_n^m -> (-1)^(n+m) c_n^m, turns a translation with
//   t_z < 0 into the one with |t_z|: translations are classed by (|t_z|, rho),
//   34 classes for the 316 far-field offsets, and one class shares W and C.
//
// One block takes a group of destination boxes, one right-hand side and one of
// its channels (all three at small orders), and walks the group's pairs class by
// class, eight at a time.  A tile's vectors are the sixteen real columns (pair,
// re/im) of an LDS buffer with one row per coefficient.  Each wavefront owns a
// fixed share of the blocks of W^n and C^m, and holds their fragments in
// registers for as long as the class lasts: a phase is LDS reads, 16x16x4 MFMA
// steps and LDS writes in place at compile-time addresses, and the next class's
// fragments arrive behind the phases that do not need them.  The results are
// added to the group's expansions in LDS, each destination's pairs in one fixed
// order, so sums do not depend on timing.
//
// What bounds it: the matrix cores, whose 16-row steps find blocks of 1 to p rows
// (57% of the steps' work is useful at p = 17, 40% at p = 12), and the opening and
// closing of a tile, about as long again.  583,336 S|R pairs (the 753k-node
// ellipsoid's leaves): FP64 p = 17 23.1 -> 6.9 ms, of which 2.5 ms are MFMA steps
// at full rate; FP32 p = 12 2.75 -> 1.81 ms (0.6 ms); the torus's 101,536 at FP64
// p = 23 6.7 -> 3.1 ms (0.85 ms).  The version before gave each pair to one
// wavefront's vector units, its tables read through L2 per pair.  Measured and
// dropped here: a wavefront per tile with no barriers and the sums in cache
// instead of LDS (16 ms where this takes 8), three channels per block at p = 12
// (2.2 ms), 8 wavefronts at p = 12 (2.1 ms), loading sources a tile ahead (1.9 ms).
#pragma once

#include <utility>

#include "rcs.h"

namespace fmb {

constexpr int RCS_MAXLEV = 10;

// one set of a launch
struct RcsLev {
    int blk0, ngroups, zsplit, tg, ncls, ps, pd, phs, nbox, accumulate;
    const int32_t *gcls, *cdist;
    const int2 *ent;
    const void *ph, *W, *C, *S;
    void *D, *part;
};

struct RcsArgs {
    int nlev, nrhs_max;
    RcsLev lev[RCS_MAXLEV];
};

template <typename T>
struct Mma;
// 16x16x4: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; register q of
// lane l holds D[l / 16 + 4 q][l % 16] in FP64.  FP32 puts row 4 (l / 16) + q there:
// its fragments list the rows in an order that gives the FP64 placement.
template <>
struct Mma<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(double a, double b, v4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};
template <>
struct Mma<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(float a, float b, v4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

// x of the neighbouring column (re <-> im), with mask xored into its sign
__device__ __forceinline__ float rcs_swap(float x, int mask) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true) ^ mask);
}
__device__ __forceinline__ double rcs_swap(double x, int mask) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0xB1, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0xB1, 0xF, 0xF, true) ^ mask;
    return __hiloint2double(hi, lo);
}

// barrier that orders LDS accesses only: fragment loads in flight stay in flight
__device__ __forceinline__ void rcs_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// rotation block of degree N, parity PAR (B = N + 1 - PAR rows from N^2 + PAR (N + 1)), in place.  Register q of a lane
// is row l / 16 + 4 q of the block, as input step and as output: only the last step has rows to leave out.
template <typename T, int P, int NC, int N, int PAR>
__device__ __forceinline__ void rcs_rot(T *buf, const T *f, int lane) {
    typedef typename Mma<T>::v4 v4;
    constexpr int B = N + 1 - PAR, KS = (B + 3) / 4, RT = (B + 15) / 16;
    const bool last = B % 4 == 0 || (lane >> 4) < B - 4 * (KS - 1);
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
        T *at = buf + (nc * P * P + N * N + PAR * (N + 1)) * 16 + lane;
        T x[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) x[k] = at[k * 64];
        x[KS - 1] = last ? x[KS - 1] : T(0);
        v4 acc[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[i] = v4{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int i = 0; i < RT; ++i) acc[i] = Mma<T>::mma(f[i * KS + k], x[k], acc[i]);
#pragma unroll
        for (int k = 0; k < KS; ++k)
            if (k < KS - 1 || last) at[k * 64] = acc[k / 4][k % 4];
    }
}

// axial shift of order |m| = AM, both parities (rows n^2 + par n + AM), in place; re = Cr xr - Ci xi,
// im = Cr xi + Ci xr: the second product takes the neighbouring column, negated for re
template <typename T, int P, int NC, int AM>
__device__ __forceinline__ void rcs_shift(T *buf, const T *f, int lane) {
    typedef typename Mma<T>::v4 v4;
    constexpr int B = P - AM, KS = (B + 3) / 4, RT = (B + 15) / 16;
    const int kq = lane >> 4, mask = (lane & 1) ? 0 : (int)0x80000000;
    const bool last = B % 4 == 0 || kq < B - 4 * (KS - 1);
#pragma unroll
    for (int par = 0; par < (AM ? 2 : 1); ++par)
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
            // row of n = AM + kq + 4 k: (AM + 4 k)^2 + par (AM + 4 k) + AM + kq (kq + 2 AM + 8 k + par)
            int off[KS];
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                constexpr int a = AM;
                const int c = a + 4 * k;
                off[k] = (nc * P * P + c * c + par * c + a) * 16 + kq * (kq + 2 * c + par) * 16 + (lane & 15);
            }
            T x[KS], y[KS];
#pragma unroll
            for (int k = 0; k < KS - 1; ++k) x[k] = buf[off[k]];
            x[KS - 1] = buf[last ? off[KS - 1] : 0];
            x[KS - 1] = last ? x[KS - 1] : T(0);
#pragma unroll
            for (int k = 0; k < KS; ++k) y[k] = rcs_swap(x[k], mask);
            v4 acc[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) acc[i] = v4{0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < KS; ++k) {
#pragma unroll
                for (int i = 0; i < RT; ++i) acc[i] = Mma<T>::mma(f[i * KS + k], x[k], acc[i]);
#pragma unroll
                for (int i = 0; i < RT; ++i) acc[i] = Mma<T>::mma(f[(RT + i) * KS + k], y[k], acc[i]);
            }
#pragma unroll
            for (int k = 0; k < KS; ++k)
                if (k < KS - 1 || last) buf[off[k]] = acc[k / 4][k % 4];
        }
}

// wavefront WV's share of the rotation blocks / axial shifts
template <typename T, int P, int WAVES, int NC, int WV, int I>
__device__ __forceinline__ void rcs_rot_item(T *buf, const T *f, int lane) {
    constexpr RcsMap M = rcs_map(P, WAVES);
    if constexpr (M.rw[I] == WV) rcs_rot<T, P, NC, I / 2, I % 2>(buf, f + M.ro[I], lane);
}
template <typename T, int P, int WAVES, int NC, int WV, int... I>
__device__ __forceinline__ void rcs_rot_wave(T *buf, const T *f, int lane, std::integer_sequence<int, I...>) {
    (rcs_rot_item<T, P, WAVES, NC, WV, I>(buf, f, lane), ...);
}
template <typename T, int P, int WAVES, int NC, int WV, int I>
__device__ __forceinline__ void rcs_shift_item(T *buf, const T *f, int lane) {
    constexpr RcsMap M = rcs_map(P, WAVES);
    if constexpr (M.sw[I] == WV) rcs_shift<T, P, NC, I>(buf, f + M.so[I], lane);
}
template <typename T, int P, int WAVES, int NC, int WV, int... I>
__device__ __forceinline__ void rcs_shift_wave(T *buf, const T *f, int lane, std::integer_sequence<int, I...>) {
    (rcs_shift_item<T, P, WAVES, NC, WV, I>(buf, f, lane), ...);
}
template <typename T, int P, int WAVES, int NC, int WV = 0>
__device__ __forceinline__ void rcs_rotate(int wave, T *buf, const T *f, int lane) {
    if (WV == 0) asm volatile("" : "+v"(lane));      // addresses are recomputed per tile, not kept in registers
    if (wave == WV) rcs_rot_wave<T, P, WAVES, NC, WV>(buf, f, lane, std::make_integer_sequence<int, 2 * P>());
    else if constexpr (WV + 1 < WAVES) rcs_rotate<T, P, WAVES, NC, WV + 1>(wave, buf, f, lane);
}
template <typename T, int P, int WAVES, int NC, int WV = 0>
__device__ __forceinline__ void rcs_axial(int wave, T *buf, const T *f, int lane) {
    if (WV == 0) asm volatile("" : "+v"(lane));
    if (wave == WV) rcs_shift_wave<T, P, WAVES, NC, WV>(buf, f, lane, std::make_integer_sequence<int, P>());
    else if constexpr (WV + 1 < WAVES) rcs_axial<T, P, WAVES, NC, WV + 1>(wave, buf, f, lane);
}

// (n, m) of the t-th pair 0 <= m <= n, packed n << 8 | m
__device__ inline int rcs_nm(int t) {
    int n = (int)((sqrtf(8.f * t + 1.f) - 1.f) * 0.5f);
    while (n * (n + 1) / 2 > t) --n;
    while ((n + 1) * (n + 2) / 2 <= t) ++n;
    return n << 8 | (t - n * (n + 1) / 2);
}

__device__ __forceinline__ float rcs_flip(float x, int mask) { return __int_as_float(__float_as_int(x) ^ mask); }
__device__ __forceinline__ double rcs_flip(double x, int mask) {
    return __hiloint2double(__double2hiint(x) ^ mask, __double2loint(x));
}

template <typename T, int P, int NC, int WAVES, int MINW>
__global__ void __launch_bounds__(WAVES * 64, MINW) k_rcs(RcsArgs A) {
    extern __shared__ __align__(16) unsigned char rcs_smem[];
    constexpr RcsMap M = rcs_map(P, WAVES);
    constexpr int TPB = WAVES * 64, IS = TPB / RCS_TILE, NI = P * (P + 1) / 2, IT = (NI + IS - 1) / IS;
    constexpr int PLANE = P * P * 16;
    typedef cx<T> C;
    int li = 0;
    while (li + 1 < A.nlev && A.lev[li + 1].blk0 <= (int)blockIdx.x) ++li;
    const RcsLev &V = A.lev[li];
    int loc = blockIdx.x - V.blk0;
    const int g = loc % V.ngroups;
    loc /= V.ngroups;
    const int z = loc % V.zsplit, col = loc / V.zsplit;
    const int r = col / (3 / NC), ch = NC == 3 ? 0 : col % 3;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ps = V.ps, pd = V.pd, S2 = ps * ps, D2 = pd * pd;
    T *buf = reinterpret_cast<T *>(rcs_smem);
    // a tile's phases [m][pair], two of them: a wavefront may open the next tile while another closes this one
    C *phs = reinterpret_cast<C *>(buf + NC * PLANE + 64);
    C *acc = phs + 2 * P * RCS_TILE;                                    // [tg][NC][D2]
    const int b0 = g * V.tg, nb = min(V.tg, V.nbox - b0);
    C *Dg = (C *)V.D + (((int64_t)b0 * A.nrhs_max + r) * 3 + ch) * D2;
    const int64_t dbox = (int64_t)A.nrhs_max * 3 * D2;
    for (int t = tid; t < nb * NC * D2; t += TPB) {
        const int b = t / (NC * D2), e = t - b * NC * D2;
        acc[t] = V.accumulate ? Dg[b * dbox + e] : mk(T(0), T(0));
    }
    // class bounds and axial tables, a class per lane (ncls < 64)
    const int bound = V.gcls[(int64_t)g * (V.ncls + 1) + min(lane, V.ncls)];
    const int cdist = V.cdist[min(lane, V.ncls - 1)];
    // this thread's pair of a tile and its coefficients (n, +-m): opening and closing read and write the same LDS cells,
    // and a coefficient's sums stay within one wavefront
    const int j = tid & (RCS_TILE - 1);
    int mn_[IT], up_[IT];                        // m | n << 12, n^2 + n + m
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int nm = rcs_nm(min((tid >> 3) + i * IS, NI - 1)), n = nm >> 8, m = nm & 255;
        mn_[i] = m | n << 12;
        up_[i] = n * n + n + m;
    }
    // with many coefficients per thread, what follows from these is recomputed per tile, not kept in registers
    auto renew = [&]() {
        if (IT >= 4 || sizeof(T) == 8) {
#pragma unroll
            for (int i = 0; i < IT; ++i) asm volatile("" : "+v"(mn_[i]), "+v"(up_[i]));
        }
    };
    // n^2 + n - m, and the LDS cell of the even part, (n^2 + m) 16 + 2 j
    auto dn_of = [&](int i) { return up_[i] - 2 * (mn_[i] & 255); };
    auto at_of = [&](int i) { return up_[i] * 16 - (mn_[i] >> 8) + 2 * j; };
    // tiles: class by class, RCS_TILE pairs at a time; with zsplit every zsplit-th
    int cls = 0, q = __builtin_amdgcn_readlane(bound, 0), qe = __builtin_amdgcn_readlane(bound, 1), skip = z;
    auto settle = [&]() {
        for (;;) {
            while (q >= qe && cls < V.ncls) {
                if (++cls == V.ncls) return;
                q = qe;
                qe = __builtin_amdgcn_readlane(bound, cls + 1);
            }
            if (skip == 0) break;
            --skip;
            q += RCS_TILE;
        }
        skip = V.zsplit;
    };
    settle();
    T wf[M.rmax], cf[M.smax];
    auto fetch_w = [&](int c) {
        const T *F = (const T *)V.W + ((int64_t)c * WAVES + wave) * M.rmax * 64 + lane;
#pragma unroll
        for (int i = 0; i < M.rmax; ++i) wf[i] = F[i * 64];
    };
    auto fetch_c = [&](int c) {
        const T *F = (const T *)V.C + ((int64_t)__builtin_amdgcn_readlane(cdist, c) * WAVES + wave) * M.smax * 64 + lane;
#pragma unroll
        for (int i = 0; i < M.smax; ++i) cf[i] = F[i * 64];
    };
    int2 en = make_int2(0, 0);
    if (cls < V.ncls) {
        if (j < qe - q) en = V.ent[q + j];
        fetch_w(cls);
        fetch_c(cls);
    }
    rcs_sync();
    for (int tile = 0; cls < V.ncls; ++tile) {
        C *pht = phs + (tile & 1) * P * RCS_TILE;
        const int cnt = min(RCS_TILE, qe - q);
        renew();
        const int pair = en.y, flip = pair << 23;              // bit 8 of a pair: reflect, here as a sign
        {
            // phases, reflection and the even/odd combinations of the sources; columns past the last pair hold
            // whatever box 0 gives and are never read
            const C *src = (const C *)V.S + (((int64_t)en.x * A.nrhs_max + r) * 3 + ch) * S2;
            const C *pj = (const C *)V.ph + (int64_t)(pair >> 13) * V.phs;
            C f[IT], xu[IT][NC], xd[IT][NC];
#pragma unroll
            for (int i = 0; i < IT; ++i)
#pragma unroll
                for (int nc = 0; nc < NC; ++nc) {
                    xu[i][nc] = xd[i][nc] = mk(T(0), T(0));
                    if (mn_[i] >> 12 < ps) {         // degrees from ps to P: zero
                        xu[i][nc] = src[nc * S2 + up_[i]];
                        xd[i][nc] = src[nc * S2 + dn_of(i)];
                    }
                }
#pragma unroll
            for (int i = 0; i < IT; ++i) f[i] = pj[min(mn_[i] & 255, V.phs - 1)];   // e^{i m phi} / sqrt 2, 1 / 2 at m = 0
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                // closing: (-1)^m and, reflected, (-1)^(n + m), of which (-1)^m goes with the phase here
                const int em = mn_[i] << 31, en_ = mn_[i] << 19 & (int)0x80000000;
                if ((mn_[i] >> 12) == (mn_[i] & 255)) {
                    const int o2 = em ^ (flip & em);
                    pht[(mn_[i] & 255) * RCS_TILE + j] = mk(rcs_flip(f[i].re, o2), rcs_flip(f[i].im, o2));
                }
                const int odd = flip & (em ^ en_) & (int)0x80000000;
                f[i] = mk(rcs_flip(f[i].re, odd), rcs_flip(f[i].im, odd));
                T *o = buf + at_of(i);
#pragma unroll
                for (int nc = 0; nc < NC; ++nc) {
                    const C s = xu[i][nc] + xd[i][nc], d = xu[i][nc] - xd[i][nc];
                    if (i < IT - 1 || (tid >> 3) + i * IS < NI) {
                        *(C *)(o + nc * PLANE) = mk(f[i].re * s.re - f[i].im * d.im, f[i].re * s.im + f[i].im * d.re);
                        if (mn_[i] & 255)
                            *(C *)(o + nc * PLANE + (mn_[i] >> 8)) =
                                mk(f[i].re * d.re - f[i].im * s.im, f[i].re * d.im + f[i].im * s.re);
                    }
                }
            }
        }
        // the next tile
        const int cls0 = cls;
        q += RCS_TILE;
        --skip;
        settle();
        const bool more = cls < V.ncls, turn = more && cls != cls0;
        en = make_int2(0, 0);
        if (more && j < qe - q) en = V.ent[q + j];
        rcs_sync();
        rcs_rotate<T, P, WAVES, NC>(wave, buf, wf, lane);
        rcs_sync();
        rcs_axial<T, P, WAVES, NC>(wave, buf, cf, lane);
        if (turn) fetch_c(cls);
        rcs_sync();
        rcs_rotate<T, P, WAVES, NC>(wave, buf, wf, lane);
        if (turn) fetch_w(cls);
        rcs_sync();
        // closing phases and sums; pairs of the tile that share a destination take turns, in list order
        renew();
        const int turnof = (pair >> 9) & 15;
        C *ac = acc + (pair & 255) * NC * D2;
        for (int k = 0;; ++k) {
            if (j < cnt && turnof == k) {
#pragma unroll
                for (int i = 0; i < IT; ++i) {
                    if ((i < IT - 1 || (tid >> 3) + i * IS < NI) && mn_[i] >> 12 < pd) {
                        const C f = pht[(mn_[i] & 255) * RCS_TILE + j];
                        const int odd = flip & mn_[i] << 19 & (int)0x80000000;
                        const C h = mk(rcs_flip(f.re, odd), rcs_flip(f.im, odd));
                        const T *o = buf + at_of(i);
#pragma unroll
                        for (int nc = 0; nc < NC; ++nc) {
                            C *a = ac + nc * D2;
                            const int dn = dn_of(i);
                            const C E = *(const C *)(o + nc * PLANE), Oz = *(const C *)(o + nc * PLANE + (mn_[i] >> 8));
                            const bool m0 = !(mn_[i] & 255);
                            const C O = m0 ? E : Oz;
                            const C s = E + O, d = E - O, u = a[up_[i]], v = a[dn];
                            a[up_[i]] = mk(u.re + h.re * s.re + h.im * s.im, u.im + h.re * s.im - h.im * s.re);
                            if (!m0) a[dn] = mk(v.re + h.re * d.re - h.im * d.im, v.im + h.re * d.im + h.im * d.re);
                        }
                    }
                }
            }
            if (!__any(j < cnt && turnof > k)) break;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    rcs_sync();
    C *out = Dg;
    if (V.zsplit > 1) out = (C *)V.part + ((((int64_t)z * V.nbox + b0) * A.nrhs_max + r) * 3 + ch) * D2;
    for (int t = tid; t < nb * NC * D2; t += TPB) {
        const int b = t / (NC * D2), e = t - b * NC * D2;
        out[b * dbox + e] = acc[t];
    }
}

// block shape of order P: wavefronts, channels per block, blocks that the registers should leave room for on a CU
template <typename T>
constexpr int rcs_waves(int P) { return sizeof(T) == 4 ? (P <= 12 ? 4 : 8) : (P <= 8 ? 4 : 8); }
template <typename T>
constexpr int rcs_nc(int P) { return sizeof(T) == 4 && P <= 9 ? 3 : 1; }

template <typename T, int P>
void rcs_launch(const RcsArgs &A, unsigned blocks, size_t lds, hipStream_t s) {
    constexpr int W = rcs_waves<T>(P);
    constexpr int MINW = P <= 18 ? 4 : 2;   // wavefronts per SIMD
    auto kern = k_rcs<T, P, rcs_nc<T>(P), W, MINW>;
    if (lds > 64 * 1024)
        FMB_CHECK_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)RCS_LDS_MAX));
    kern<<<blocks, W * 64, lds, s>>>(A);
    FMB_LAUNCH_CHECK();
}

// the orders that rcs_order gives
#define RCS_ORDERS32_LO(X) X(float, 2) X(float, 3) X(float, 4) X(float, 5) X(float, 6) X(float, 7) X(float, 8) X(float, 9) \
    X(float, 10) X(float, 11) X(float, 12) X(float, 14) X(float, 16)
#define RCS_ORDERS32_MID(X) X(float, 17) X(float, 18) X(float, 20) X(float, 21) X(float, 22) X(float, 23) X(float, 24)
#define RCS_ORDERS32_HI(X) X(float, 26) X(float, 28) X(float, 30) X(float, 32)
#define RCS_ORDERS64_LO(X) X(double, 2) X(double, 3) X(double, 4) X(double, 5) X(double, 6) X(double, 7) X(double, 8) \
    X(double, 9) X(double, 10) X(double, 11) X(double, 12) X(double, 14) X(double, 16)
#define RCS_ORDERS64_MID(X) X(double, 17) X(double, 18) X(double, 20)
#define RCS_ORDERS64_HI(X) X(double, 21) X(double, 22) X(double, 23) X(double, 24)
#define RCS_ORDERS32(X) RCS_ORDERS32_LO(X) RCS_ORDERS32_MID(X) RCS_ORDERS32_HI(X)
#define RCS_ORDERS64(X) RCS_ORDERS64_LO(X) RCS_ORDERS64_MID(X) RCS_ORDERS64_HI(X)
#define RCS_INSTANTIATE(T, P) template void rcs_launch<T, P>(const RcsArgs &, unsigned, size_t, hipStream_t);

}  // namespace fmb
