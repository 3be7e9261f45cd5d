// Translations by rotation, coaxial shift and rotation back on the matrix
// cores: what a plan keeps for one translation set, and its interface.
#pragma once

#include <complex>
#include <vector>

#include "common.h"

namespace fmb {

constexpr int RCS_PMAX32 = 32, RCS_PMAX64 = 24;     // largest order of a set (source or destination) per precision
constexpr int RCS_TILE = 8;                         // pairs of one class that run through the matrix cores together
constexpr size_t RCS_LDS_MAX = 160 * 1024 - 1024;   // beside the kernel's own arrays

// The order whose kernel serves order p: all to 12, then every second, and 17, 21 and 23.  17 and 23 are the order rule's
// for 1e-6 and 1e-8, 21 is next above the leaves of bodies many wavelengths across.  A product on a kernel of their own
// against the next larger (torus 60,000 nodes, ms): FP64 17 2.55 / 3.19, 21 3.99 / 4.22, 23 4.96 / 5.18; FP32 1.28 / 1.36,
// 1.91 / 2.04, 2.99 / 3.13.  13, 15, 19 and the odd ones above 24 have not been measured.
constexpr int rcs_order(int p) {
    return p <= 12 || p == 17 || p == 21 || p == 23 ? (p < 2 ? 2 : p) : (p + 1) / 2 * 2;
}

// Share-out of order P's work over W wavefronts, largest items to the least loaded.  Rotation item 2 n + par:
// parity block of degree n; shift item m.  Each has its wavefront and its first fragment there.
struct RcsMap {
    int rw[64] = {}, ro[64] = {}, sw[32] = {}, so[32] = {};
    int rmax = 0, smax = 0;          // fragments of the fullest wavefront
};
constexpr int rcs_frags(int b) { return (b + 15) / 16 * ((b + 3) / 4); }
constexpr RcsMap rcs_map(int P, int W) {
    RcsMap M;
    int cost[16] = {}, used[16] = {};
    for (int b = P; b >= 1; --b)
        for (int par = 0; par < 2; ++par) {
            const int n = b - 1 + par;
            if (n >= P) continue;
            int w = 0;
            for (int i = 1; i < W; ++i)
                if (cost[i] < cost[w]) w = i;
            M.rw[2 * n + par] = w;
            M.ro[2 * n + par] = used[w];
            used[w] += rcs_frags(b);
            cost[w] += 4 * rcs_frags(b) + 3;
            if (used[w] > M.rmax) M.rmax = used[w];
        }
    M.rw[1] = -1;                    // degree 0 has no odd combination
    for (int i = 0; i < 16; ++i) cost[i] = used[i] = 0;
    // order 0 has one parity: it comes where its weight puts it
    for (int k = 0; k < P; ++k) {
        const int h = P / 2, m = k < h ? k + 1 : (k == h ? 0 : k);
        int w = 0;
        for (int i = 1; i < W; ++i)
            if (cost[i] < cost[w]) w = i;
        M.sw[m] = w;
        M.so[m] = used[w];
        used[w] += 2 * rcs_frags(P - m);
        cost[w] += (m ? 2 : 1) * (8 * rcs_frags(P - m) + 4);
        if (used[w] > M.smax) M.smax = used[w];
    }
    return M;
}

// One translation set: the S|R pairs of a level, or its S|S or R|R.  Destination
// boxes form groups of tg consecutive boxes; a group's pairs are sorted by class
// (translations that share their polar angle up to a reflection in z, and their
// length: one rotation and one axial table each).
struct RcsSet {
    bool on = false;
    int ps = 0, pd = 0, P = 0;    // source and destination orders, the kernel's order
    int ncls = 0, tg = 1, ngroups = 0, zsplit = 1, nc = 1, waves = 4;
    int64_t nbox = 0;
    DevBuf gcls;                  // i32[ngroups][ncls + 1] bounds of each class's pairs
    DevBuf ent;                   // i32[npairs][2]: source box; destination, reflection, turn, direction (k_rcs_lists)
    DevBuf W, C;                  // matrix-core fragments: [ncls][waves][rmax][64], [distances][waves][smax][64]
    DevBuf ph;                    // e^{i m phi} / sqrt 2 (1 / 2 at m = 0) of each direction, phs entries apart
    int phs = 0;
    DevBuf cdist;                 // i32[ncls] distance of each class (none: one distance)
    DevBuf part;                  // zsplit > 1: [zsplit][nbox][nrhs_max][3][pd^2] partial sums
    size_t lds = 0;
    size_t bytes() const {
        return gcls.bytes + ent.bytes + W.bytes + C.bytes + ph.bytes + cdist.bytes + part.bytes;
    }
};

// one set of a run: D (=, or += with accumulate) its translations of S
struct RcsJob {
    const RcsSet *set;
    const void *S;
    void *D;
    int accumulate;
};

enum RcsKind { RCS_SR, RCS_SS, RCS_RR };
// orders and block shape, before anything else of a set is built
void rcs_shape(RcsSet &R, int ps, int pd, int64_t nbox, bool f64, RcsKind kind);
// fragments of one table in the kernel's layout: W as rotation_table gives it for degrees n < p (p = max(ps, pd)),
// C as coax_table (pd x ps)
template <typename T>
void rcs_rotation(const RcsSet &R, const double *W, T *out);
template <typename T>
void rcs_coaxial(const RcsSet &R, const std::complex<double> *C, T *out);
int64_t rcs_wsize(const RcsSet &R);
int64_t rcs_csize(const RcsSet &R);
// npairs pairs: destination b's are ofs[b] .. ofs[b + 1] (b itself without ofs), from sources src[e] (e without src) in
// directions dir[e] + dir_add, of class cls_of[direction] & 255, reflected if bit 8 is set; cdist: each class's axial table
void rcs_build(RcsSet &R, int64_t npairs, const DevBuf *ofs, const DevBuf *src, const DevBuf &dir, int dir_add,
               const std::vector<int32_t> &cls_of, const std::vector<int32_t> &cdist, hipStream_t s);
void rcs_split(RcsSet **sets, int nsets, bool f64, int nrhs_max);
// returns the kernels it launched
template <typename T>
int rcs_run(const RcsJob *jobs, int njobs, int nrhs, int nrhs_max, hipStream_t s);

}  // namespace fmb
