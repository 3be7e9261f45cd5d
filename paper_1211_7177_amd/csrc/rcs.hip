// Translations on the matrix cores (rcs_kernel.h): plan-time lists and tables, and the launches.
#include <algorithm>
#include <cmath>
#include <complex>

#include "plan.h"
#include "rcs_kernel.h"

namespace fmb {

namespace {

// destinations of sets whose tiles were split over zsplit blocks: the partial sums in order, all sets of a launch
struct SumArgs {
    int nset, nrhs, nrhs_max;
    int64_t first[RCS_MAXLEV + 1];
    int zsplit[RCS_MAXLEV], blk[RCS_MAXLEV];
    const void *part[RCS_MAXLEV];
    void *D[RCS_MAXLEV];
};
template <typename T>
__global__ void k_rcs_sum(SumArgs A) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= A.first[A.nset]) return;
    int l = 0;
    while (A.first[l + 1] <= i) ++l;
    i -= A.first[l];
    const int blk = A.blk[l];
    const int64_t per = (int64_t)A.nrhs * blk, box = i / per, e = i - box * per;
    const int64_t st = (A.first[l + 1] - A.first[l]) / per * A.nrhs_max * blk;
    const cx<T> *p = (const cx<T> *)A.part[l] + box * A.nrhs_max * blk + e;
    cx<T> s = p[0];
    for (int z = 1; z < A.zsplit[l]; ++z) s += p[z * st];
    ((cx<T> *)A.D[l])[box * A.nrhs_max * blk + e] = s;
}

// Pairs of group g sorted by (class, how many of the destination's pairs of this class came before, destination), one
// wavefront per group: a tile then meets most destinations once.  Destination b's pairs are ofs[b] .. ofs[b + 1] (b
// itself without ofs), with sources src[e] (e without src) and directions dir[e] + dir_add.  A pair is packed as
// destination in group | reflect << 8 | earlier pairs of its tile with its destination << 9 | direction << 13.
constexpr int LIST_TG = 16, LIST_CLS = 40, LIST_OCC = 16;

__global__ void __launch_bounds__(64) k_rcs_lists(const int32_t *__restrict__ ofs, const int32_t *__restrict__ src,
                                                  const int32_t *__restrict__ dir, int dir_add,
                                                  const int32_t *__restrict__ cls_of, int nbox, int tg, int ncls,
                                                  int32_t *__restrict__ gcls, int2 *__restrict__ ent) {
    __shared__ int seen[LIST_TG * LIST_CLS], pos[LIST_CLS * LIST_OCC], box_end[LIST_TG];
    const int g = blockIdx.x, lane = threadIdx.x;
    const int b0 = g * tg, b1 = min(nbox, b0 + tg);
    const int e0 = ofs ? ofs[b0] : b0, e1 = ofs ? ofs[b1] : b1;
    int32_t *gc = gcls + (int64_t)g * (ncls + 1);
    for (int t = lane; t < b1 - b0; t += 64) box_end[t] = ofs ? ofs[b0 + t + 1] : b0 + t + 1;
    for (int t = lane; t < LIST_CLS * LIST_OCC; t += 64) pos[t] = 0;
    for (int pass = 0; pass < 2; ++pass) {
        for (int t = lane; t < LIST_TG * LIST_CLS; t += 64) seen[t] = 0;
        __syncthreads();
        for (int base = e0; base < e1; base += 64) {
            const int e = base + lane;
            const bool act = e < e1;
            const int d = act ? dir[e] + dir_add : 0, cf = act ? cls_of[d] : 0, c = cf & 255;
            int b = 0;
            while (act && box_end[b] <= e) ++b;
            // lanes of the same (class, destination) before this one
            unsigned long long same = __ballot(act);
            const int key = c | b << 6;
            for (int k = 0; k < 10; ++k) {
                const unsigned long long m = __ballot((key >> k) & 1);
                same &= ((key >> k) & 1) ? m : ~m;
            }
            const int rank = __popcll(same & ((1ull << lane) - 1ull));
            const int occ = min(act ? seen[b * LIST_CLS + c] + rank : 0, LIST_OCC - 1);
            // lanes of the same (class, occurrence) before this one
            unsigned long long eq = __ballot(act);
            const int key2 = c | occ << 6;
            for (int k = 0; k < 10; ++k) {
                const unsigned long long m = __ballot((key2 >> k) & 1);
                eq &= ((key2 >> k) & 1) ? m : ~m;
            }
            const int rank2 = __popcll(eq & ((1ull << lane) - 1ull));
            const int at = act ? pos[c * LIST_OCC + occ] + rank2 : 0;
            __syncthreads();
            if (act && rank == 0) seen[b * LIST_CLS + c] += __popcll(same);
            if (act && rank2 == 0) pos[c * LIST_OCC + occ] += __popcll(eq);
            if (act && pass) ent[at] = make_int2(src ? src[e] : e, b | (cf >> 8) << 8 | d << 13);
            __syncthreads();
        }
        if (pass == 0) {
            if (lane == 0) {
                int s = e0;
                for (int c = 0; c < ncls; ++c) {
                    gc[c] = s;
                    for (int k = 0; k < LIST_OCC; ++k) {
                        const int n = pos[c * LIST_OCC + k];
                        pos[c * LIST_OCC + k] = s;
                        s += n;
                    }
                }
                gc[ncls] = s;
            }
            __syncthreads();
        }
    }
    __threadfence_block();
    __syncthreads();
    for (int c = 0; c < ncls; ++c) {
        const int q0 = gc[c], q1 = gc[c + 1];
        for (int base = q0; base < q1; base += 64) {          // 64 is a whole number of tiles
            const int q = base + lane;
            const int y = q < q1 ? ent[q].y : -1;
            int turn = 0;
            for (int k = 1; k < RCS_TILE; ++k) {
                const int o = __shfl(y, max(lane - k, 0));
                if (k <= (lane & (RCS_TILE - 1)) && (o & 255) == (y & 255)) ++turn;
            }
            if (q < q1) ent[q].y = y | turn << 9;
        }
    }
}

template <typename T>
size_t lds_of(const RcsSet &R) {
    return ((size_t)R.nc * R.P * R.P * 16 + 64 + R.P * RCS_TILE * 4 + (size_t)R.tg * R.nc * R.pd * R.pd * 2) * sizeof(T);
}

}  // namespace

void rcs_shape(RcsSet &R, int ps, int pd, int64_t nbox, bool f64, RcsKind kind) {
    R.ps = ps;
    R.pd = pd;
    R.P = rcs_order(std::max(ps, pd));
    R.nbox = nbox;
    R.nc = f64 ? rcs_nc<double>(R.P) : rcs_nc<float>(R.P);
    R.waves = f64 ? rcs_waves<double>(R.P) : rcs_waves<float>(R.P);
    // destinations per group.  S|R: 16, which fill most of a class's tiles; S|S: fewer where a level would
    // otherwise keep few blocks busy (a group's tiles run one after the other); R|R has one pair for each
    const int64_t units = nbox * (3 / R.nc);
    const int want = kind == RCS_SR   ? 16
                     : kind == RCS_SS ? (int)std::max<int64_t>(1, std::min<int64_t>(8, units / 128))
                                      : 8;
    // as many as wanted while two blocks (five small ones) share a CU's LDS, at least half of them; more than that
    // only if one block fills the CU anyway
    auto lds = [&]() { return f64 ? lds_of<double>(R) : lds_of<float>(R); };
    const size_t budget[3] = {(size_t)31 * 1024, (size_t)79 * 1024, RCS_LDS_MAX};
    R.tg = 0;
    for (int k = 0; k < 3 && R.tg == 0; ++k)
        for (int t = want; t >= (k < 2 ? (want + 1) / 2 : 1); --t) {
            R.tg = t;
            if (lds() <= budget[k]) break;
            R.tg = 0;
        }
    FMB_REQUIRE(R.tg > 0, "translation set larger than a block's LDS");
    R.lds = lds();
    R.ngroups = (int)((nbox + R.tg - 1) / R.tg);
}

int64_t rcs_wsize(const RcsSet &R) { return (int64_t)rcs_map(R.P, R.waves).rmax * R.waves * 64; }
int64_t rcs_csize(const RcsSet &R) { return (int64_t)rcs_map(R.P, R.waves).smax * R.waves * 64; }

// output row (within 16) that fragment row i of type T produces
template <typename T>
static int frag_row(int i) { return sizeof(T) == 8 ? i : i / 4 + 4 * (i % 4); }

// entry (input mi, output mo) of the parity block of degree n; w: that degree's matrix, w[(m + n) st + (m' + n)]
static double parity_entry(const double *w, int n, int par, int mi, int mo) {
    const int st = 2 * n + 1;
    const double a = w[(int64_t)(mi + n) * st + mo + n], c = w[(int64_t)(n - mi) * st + mo + n];
    if (mi == 0 && mo == 0) return a;
    if (mi == 0 || mo == 0) return std::sqrt(2.0) * a;
    return par ? a - c : a + c;
}

template <typename T>
void rcs_rotation(const RcsSet &R, const double *W, T *out) {
    const RcsMap M = rcs_map(R.P, R.waves);
    const int p = std::max(R.ps, R.pd);
    std::fill(out, out + rcs_wsize(R), T(0));
    for (int n = 0; n < p; ++n)
        for (int par = 0; par < 2; ++par) {
            if (M.rw[2 * n + par] < 0) continue;
            const int b = n + 1 - par, ks = (b + 3) / 4, rt = (b + 15) / 16;
            const double *w = W + (int64_t)n * (2 * n - 1) * (2 * n + 1) / 3;
            T *o = out + ((int64_t)M.rw[2 * n + par] * M.rmax + M.ro[2 * n + par]) * 64;
            for (int i = 0; i < rt; ++i)
                for (int k = 0; k < ks; ++k)
                    for (int l = 0; l < 64; ++l, ++o) {
                        const int mo = 16 * i + frag_row<T>(l & 15) + par, mi = 4 * k + (l >> 4) + par;
                        if (mo <= n && mi <= n) *o = (T)parity_entry(w, n, par, mi, mo);
                    }
        }
}

// (-1)^m C^m, padded with zeros to P x P
template <typename T>
void rcs_coaxial(const RcsSet &R, const std::complex<double> *C, T *out) {
    const RcsMap M = rcs_map(R.P, R.waves);
    std::fill(out, out + rcs_csize(R), T(0));
    int64_t off = 0;
    for (int m = 0; m < std::min(R.ps, R.pd); ++m) {
        const int b = R.P - m, bi = R.ps - m, bo = R.pd - m, ks = (b + 3) / 4, rt = (b + 15) / 16;
        const double sg = (m & 1) ? -1.0 : 1.0;
        T *o = out + ((int64_t)M.sw[m] * M.smax + M.so[m]) * 64;
        for (int part = 0; part < 2; ++part)
            for (int i = 0; i < rt; ++i)
                for (int k = 0; k < ks; ++k)
                    for (int l = 0; l < 64; ++l, ++o) {
                        const int q = 16 * i + frag_row<T>(l & 15), n = 4 * k + (l >> 4);
                        if (q >= bo || n >= bi) continue;
                        const std::complex<double> c = C[off + (int64_t)n * bo + q];
                        *o = (T)(sg * (part ? c.imag() : c.real()));
                    }
        off += (int64_t)bi * bo;
    }
}
template void rcs_rotation<float>(const RcsSet &, const double *, float *);
template void rcs_rotation<double>(const RcsSet &, const double *, double *);
template void rcs_coaxial<float>(const RcsSet &, const std::complex<double> *, float *);
template void rcs_coaxial<double>(const RcsSet &, const std::complex<double> *, double *);

// pairs and classes of a set (k_rcs_lists); cdist: each class's axial table
void rcs_build(RcsSet &R, int64_t npairs, const DevBuf *ofs, const DevBuf *src, const DevBuf &dir, int dir_add,
               const std::vector<int32_t> &cls_of, const std::vector<int32_t> &cdist, hipStream_t s) {
    R.on = true;
    R.ncls = (int)cdist.size();
    FMB_REQUIRE(R.ncls <= LIST_CLS && R.tg <= LIST_TG, "more translation classes or destinations than the lists hold");
    R.gcls.alloc((size_t)R.ngroups * (R.ncls + 1) * sizeof(int32_t));
    R.ent.alloc((size_t)std::max<int64_t>(1, npairs) * sizeof(int2));
    R.cdist.alloc(cdist.size() * sizeof(int32_t));
    FMB_CHECK_HIP(hipMemcpyAsync(R.cdist.p, cdist.data(), cdist.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    DevBuf co;
    co.alloc(cls_of.size() * sizeof(int32_t));
    FMB_CHECK_HIP(hipMemcpyAsync(co.p, cls_of.data(), cls_of.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    k_rcs_lists<<<(unsigned)R.ngroups, 64, 0, s>>>(ofs ? ofs->as<int32_t>() : nullptr, src ? src->as<int32_t>() : nullptr,
                                                   dir.as<int32_t>(), dir_add, co.as<int32_t>(), (int)R.nbox, R.tg,
                                                   R.ncls, R.gcls.as<int32_t>(), R.ent.as<int2>());
    FMB_LAUNCH_CHECK();
    FMB_CHECK_HIP(hipStreamSynchronize(s));
}

// Sets of few blocks split each group's tiles over zsplit of them, so that a launch over all levels holds at least
// twice what the CUs take at once (by LDS, eight blocks at most); the partial sums stay under 100 MB a set at every
// order and batch.  S|R of all levels, unsplit -> split: ring 148k FP64 p = 16 1.82 -> 1.34 ms, 26k ellipsoid FP32
// p = 12 1.0 -> 0.48 ms, sphere 3,840 nodes FP64 p = 16 (123 blocks) 0.30 ms at 6 ways, 0.28 at 8 to 16, 0.30 at 25.
// The split follows the plan's largest batch, not the call's, so that a column's sums do not depend on how many there
// are; one column on a plan for eight takes 424 us where one on a plan for one takes 342 (sphere FP64 p = 16).
void rcs_split(RcsSet **sets, int nsets, bool f64, int nrhs_max) {
    int64_t blocks = 0;
    size_t lds = 1;
    for (int i = 0; i < nsets; ++i) {
        blocks += (int64_t)sets[i]->ngroups * (3 / sets[i]->nc);
        lds = std::max(lds, sets[i]->lds);
    }
    blocks *= nrhs_max;              // a plan for batches is split for batches
    if (blocks == 0) return;
    const int64_t want = 512 * (int64_t)std::min<size_t>(8, RCS_LDS_MAX / lds);
    const int z = (int)std::min<int64_t>(32, (want + blocks - 1) / blocks);
    if (z <= 1) return;
    for (int i = 0; i < nsets; ++i) {
        RcsSet &R = *sets[i];
        R.zsplit = z;
        R.part.alloc((size_t)z * R.nbox * nrhs_max * 3 * R.pd * R.pd * (f64 ? 16 : 8));
    }
}

// ------------------------------------------------------------ launches

#define RCS_EXTERN(T, P) extern template void rcs_launch<T, P>(const RcsArgs &, unsigned, size_t, hipStream_t);
RCS_ORDERS32(RCS_EXTERN)
RCS_ORDERS64(RCS_EXTERN)
#undef RCS_EXTERN

static void launch(float, int P, const RcsArgs &A, unsigned blocks, size_t lds, hipStream_t s) {
#define RCS_CASE(T, P_) case P_: return rcs_launch<T, P_>(A, blocks, lds, s);
    switch (P) { RCS_ORDERS32(RCS_CASE) }
    throw Status{FMB_EINVAL, "no translation kernel of this order"};
}
static void launch(double, int P, const RcsArgs &A, unsigned blocks, size_t lds, hipStream_t s) {
    switch (P) { RCS_ORDERS64(RCS_CASE) }
#undef RCS_CASE
    throw Status{FMB_EINVAL, "no translation kernel of this order"};
}

// Consecutive jobs of one order go out as one launch.  A launch holds less than 2^32 threads: wider batches run in slices.
template <typename T>
int rcs_run(const RcsJob *jobs, int njobs, int nrhs, int nrhs_max, hipStream_t s) {
    int nk = 0;
    for (int a = 0; a < njobs;) {
        const RcsSet &F = *jobs[a].set;
        int b = a, slice = nrhs;
        int64_t per = 0;                  // threads of one right-hand side
        for (; b < njobs && b - a < RCS_MAXLEV; ++b) {
            const RcsSet &R = *jobs[b].set;
            if (R.P != F.P) break;
            per += (int64_t)R.ngroups * R.zsplit * (3 / R.nc) * R.waves * 64;
        }
        FMB_REQUIRE(per < (int64_t)1 << 32, "too many translation blocks");
        if (per) slice = (int)std::min<int64_t>(slice, (((int64_t)1 << 32) - 1) / per);
        for (int r0 = 0; r0 < nrhs; r0 += slice) {
            RcsArgs A{};
            A.nrhs_max = nrhs_max;
            A.nlev = b - a;
            const int nr = std::min(slice, nrhs - r0);
            size_t lds = 0;
            int64_t blocks = 0;
            for (int i = a; i < b; ++i) {
                const RcsSet &R = *jobs[i].set;
                RcsLev &V = A.lev[i - a];
                V.blk0 = (int)blocks;
                V.ngroups = R.ngroups;
                V.zsplit = R.zsplit;
                V.tg = R.tg;
                V.ncls = R.ncls;
                V.ps = R.ps;
                V.pd = R.pd;
                V.phs = R.phs;
                V.nbox = (int)R.nbox;
                V.accumulate = jobs[i].accumulate;
                V.gcls = R.gcls.as<int32_t>();
                V.ent = R.ent.as<int2>();
                V.ph = R.ph.p;
                V.W = R.W.p;
                V.C = R.C.p;
                V.cdist = R.cdist.as<int32_t>();
                V.S = (const cx<T> *)jobs[i].S + (int64_t)r0 * 3 * R.ps * R.ps;
                V.D = (cx<T> *)jobs[i].D + (int64_t)r0 * 3 * R.pd * R.pd;
                V.part = R.part.p;
                blocks += (int64_t)R.ngroups * R.zsplit * (3 / R.nc) * nr;
                lds = std::max(lds, R.lds);
            }
            if (blocks == 0) continue;
            launch(T(0), F.P, A, (unsigned)blocks, lds, s);
            ++nk;
            SumArgs Z{};
            Z.nrhs = nr;
            Z.nrhs_max = nrhs_max;
            for (int i = a; i < b; ++i) {
                const RcsSet &R = *jobs[i].set;
                if (R.zsplit == 1) continue;
                const int l = Z.nset++;
                Z.zsplit[l] = R.zsplit;
                Z.blk[l] = 3 * R.pd * R.pd;
                Z.part[l] = R.part.p;
                Z.D[l] = A.lev[i - a].D;
                Z.first[l + 1] = Z.first[l] + R.nbox * nr * Z.blk[l];
            }
            if (Z.nset) {
                k_rcs_sum<T><<<(unsigned)((Z.first[Z.nset] + 255) / 256), 256, 0, s>>>(Z);
                FMB_LAUNCH_CHECK();
                ++nk;
            }
        }
        a = b;
    }
    return nk;
}
template int rcs_run<float>(const RcsJob *, int, int, int, hipStream_t);
template int rcs_run<double>(const RcsJob *, int, int, int, hipStream_t);

}  // namespace fmb
