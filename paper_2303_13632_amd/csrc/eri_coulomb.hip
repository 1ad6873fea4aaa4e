// The adjoint's density form for screened plans: L = sum w D_ab D_cd (ab|cd)
// and its gradient from the Hermite potentials of the primitive pairs
// (codegen_coulomb.py has the scheme).
//
// Steps of a call, all on the caller's stream:
//   1. charge: H_i[t] of every primitive pair from the density;
//   2. one launch per (target order, source order): potentials V_i[t] and L;
//   3. gradient: each primitive pair's derivatives, which are Gaussian
//      products with up to two more units of angular momentum at either
//      centre, against V_i, into the slices of the gradient.
// Every quartet of the plan enters twice, once for each of its pairs, so all
// four centres are differentiated explicitly.
//
// Bound by FP64 issue in step 2 (the Boys function for small orders, R and its
// products with H for large ones).  Computing some 15 sets of integrals over
// derived shells per quartet instead took 788 ms for energy and gradient of a
// 24-atom basis (96 shells, K up to 6); this takes 9.5 ms.  Its error against
// the oracle's analytic gradient is 1.5e-14 of the largest entry on a 4- and a
// 6-atom basis.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "eri_coulomb.h"
#include "eri_internal.h"

using namespace eri_detail;

namespace {

constexpr int NCLS = 6;                                  // pair classes ss, ps, pp, ds, dp, dd
constexpr int CLS_LA[NCLS] = {0, 1, 1, 2, 2, 2}, CLS_LB[NCLS] = {0, 0, 1, 0, 1, 2};
constexpr int64_t COUL_JOBS = 8192;                      // jobs aimed at per kernel: eight wavefronts a SIMD
constexpr int COUL_CHUNK_MAX = 8192;
constexpr int64_t COUL_SLICE_DOUBLES = (int64_t)1 << 22; // gradient slices in all (32 MB)
constexpr int COUL_SLICES_MAX = 256;

inline int cls_of(int la, int lb) { return la == 0 ? 0 : la == 1 ? 1 + lb : 3 + lb; }
__host__ __device__ constexpr int nherm(int L) { return (L + 1) * (L + 2) * (L + 3) / 6; }

}  // namespace

struct eri_coul_state {
    int64_t prim0[NCLS + 1] = {};        // first primitive pair of each class
    int64_t rec0[NCLS] = {}, pot0[NCLS] = {};
    int64_t n_rec = 0, n_pot = 0;
    int64_t job0[26] = {};               // jobs of kernel (lt, ls) at 5 lt + ls
    eri_coul_job* d_jobs = nullptr;
    eri_coul_range* d_ranges = nullptr;
    int32_t* d_prim_pair = nullptr;
    int64_t* d_bf = nullptr;
    int64_t* d_poff = nullptr;
    double* d_rec = nullptr;
    double* d_pot = nullptr;
    double* d_energy = nullptr;          // per job (high, low)
    double* d_part = nullptr;
    int64_t nbf = 0, n_grad = 0;
    int n_slices = 1;
};

void eri_coul_free(eri_coul_state* s)
{
    if (!s) return;
    void* ptrs[] = {s->d_jobs, s->d_ranges, s->d_prim_pair, s->d_bf, s->d_poff, s->d_rec, s->d_pot, s->d_energy, s->d_part};
    for (void* x : ptrs)
        if (x) (void)hipFree(x);
    delete s;
}

namespace {

struct coul_pair_args {
    const eri_shell_pair* pairs;
    const eri_prim_pair* prims;
    const int32_t* prim_pair;
    const int64_t* bf;
    const int64_t* poff;
    const double* dens;
    int64_t nbf;
    int64_t prim0, n;        // primitive pairs of the class
    double* full;            // the class's records
    double* rec;             // and those without charges that are not finite
    const double* pot;       // the class's potentials
    int64_t pot_stride;
    double* part;
    int64_t slice_stride, ns3;
    int n_slices;
};

// Hermite expansion coefficients of one axis: x_A^i x_B^j exp(-p x_P^2) =
// sum_t E[i][j][t] Lambda_t, for i <= IA, j <= IB and i + j <= N.
template <int IA, int IB, int N>
__device__ __forceinline__ void hermite_axis(double h, double pa, double pb, double (&E)[IA + 1][IB + 1][N + 1])
{
#pragma unroll
    for (int i = 0; i <= IA; ++i)
#pragma unroll
        for (int j = 0; j <= IB; ++j) {
            if (i + j > N) continue;
#pragma unroll
            for (int t = 0; t <= N; ++t) {
                if (t > i + j) continue;
                if (i == 0 && j == 0) {
                    E[0][0][0] = 1.0;
                    continue;
                }
                const double (&S)[N + 1] = j > 0 ? E[i][j - 1] : E[i - 1][j];
                const double x = j > 0 ? pb : pa;
                const int top = i + j - 1;
                double v = t <= top ? x * S[t] : 0.0;
                if (t > 0) v = fma(h, S[t - 1], v);
                if (t + 1 <= top) v = fma((double)(t + 1), S[t + 1], v);
                E[i][j][t] = v;
            }
        }
}

// Position of (t, u, v) among the Hermites in the kernels' order.
__host__ __device__ constexpr int herm_index(int t, int u, int v)
{
    const int s = t + u + v, m = u + v;
    return s * (s + 1) * (s + 2) / 6 + m * (m + 1) / 2 + v;
}

// Exponents of component idx of a Cartesian shell (x^L first).
__device__ __forceinline__ void comp_of(int L, int idx, int (&c)[3])
{
    int m = 0;
    while ((m + 1) * (m + 2) / 2 <= idx) ++m;
    c[2] = idx - m * (m + 1) / 2;
    c[1] = m - c[2];
    c[0] = L - m;
}

template <int LA, int LB>
__global__ __launch_bounds__(64) void coul_charge_kernel(coul_pair_args A)
{
    constexpr int N = LA + LB;
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (i >= A.n) return;
    const eri_shell_pair S = A.pairs[A.prim_pair[A.prim0 + i]];
    const eri_prim_pair B = A.prims[A.prim0 + i];
    double E[3][LA + 1][LB + 1][N + 1];
#pragma unroll
    for (int x = 0; x < 3; ++x) hermite_axis<LA, LB, N>(B.hp, B.PA[x], B.alpha / B.p * S.AB[x], E[x]);
    double H[nherm(N)];
    for (int t = 0; t < nherm(N); ++t) H[t] = 0.0;
    const double w = B.kp * (S.sa != S.sb ? 2.0 : 1.0);
    const double* __restrict__ D = A.dens + A.bf[S.sa] * A.nbf + A.bf[S.sb];
    for (int ax = LA; ax >= 0; --ax)
        for (int ay = LA - ax; ay >= 0; --ay)
            for (int bx = LB; bx >= 0; --bx)
                for (int by = LB - bx; by >= 0; --by) {
                    const int az = LA - ax - ay, bz = LB - bx - by;
                    const int ia = (LA - ax) * (LA - ax + 1) / 2 + az, ib = (LB - bx) * (LB - bx + 1) / 2 + bz;
                    const double d = w * D[ia * A.nbf + ib];
                    for (int t = 0; t <= ax + bx; ++t)
                        for (int u = 0; u <= ay + by; ++u) {
                            const double xy = d * E[0][ax][bx][t] * E[1][ay][by][u];
                            for (int v = 0; v <= az + bz; ++v)
                                H[herm_index(t, u, v)] = fma(xy, E[2][az][bz][v], H[herm_index(t, u, v)]);
                        }
                }
    bool finite = true;
    for (int t = 0; t < nherm(N); ++t) finite = finite && isfinite(H[t]);
    double* __restrict__ r = A.rec + i * (4 + nherm(N));
    double* __restrict__ f = A.full + i * (4 + nherm(N));
    f[0] = B.p;
    r[0] = finite ? B.p : -B.p;
    for (int x = 0; x < 3; ++x) r[1 + x] = f[1 + x] = B.P[x];
    for (int t = 0; t <= N; ++t)
        for (int u = 0; u <= N - t; ++u)
            for (int v = 0; v <= N - t - u; ++v) {
                const int k = herm_index(t, u, v);
                f[4 + k] = (t + u + v) & 1 ? -H[k] : H[k];
                r[4 + k] = finite ? f[4 + k] : 0.0;
            }
}
// One thread per primitive pair and pair of Cartesian components (blockIdx.y):
// one thread for all components left a d-d pair's 36 of them in series over
// few threads (1.5 ms for the 440 primitive pairs of a 24-atom basis).
template <int LA, int LB>
__global__ __launch_bounds__(64) void coul_gradient_kernel(coul_pair_args A)
{
    constexpr int N = LA + LB + 2, NB = (LB + 1) * (LB + 2) / 2;
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (i >= A.n) return;
    const int ia = blockIdx.y / NB, ib = blockIdx.y % NB;
    const eri_shell_pair S = A.pairs[A.prim_pair[A.prim0 + i]];
    const eri_prim_pair B = A.prims[A.prim0 + i];
    double E[3][LA + 3][LB + 3][N + 1];
#pragma unroll
    for (int x = 0; x < 3; ++x) hermite_axis<LA + 2, LB + 2, N>(B.hp, B.PA[x], B.alpha / B.p * S.AB[x], E[x]);
    const double* __restrict__ V = A.pot + i;
    // potential of the product of x_A^a x_B^b over the axes
    auto at = [&](int ax, int ay, int az, int bx, int by, int bz) {
        double s = 0.0;
        for (int t = 0; t <= ax + bx; ++t)
            for (int u = 0; u <= ay + by; ++u) {
                const double xy = E[0][ax][bx][t] * E[1][ay][by][u];
                for (int v = 0; v <= az + bz; ++v)
                    s = fma(xy * E[2][az][bz][v], V[herm_index(t, u, v) * A.pot_stride], s);
            }
        return s;
    };
    int a[3], b[3];
    comp_of(LA, ia, a);
    comp_of(LB, ib, b);
    // L is quadratic in the charges: twice the derivative of one factor
    const double d = 2.0 * B.kp * (S.sa != S.sb ? 2.0 : 1.0) * A.dens[(A.bf[S.sa] + ia) * A.nbf + A.bf[S.sb] + ib];
    const double ta = 2.0 * B.alpha, tb = 2.0 * B.beta;
    const double s0 = at(a[0], a[1], a[2], b[0], b[1], b[2]);
    double ea = (0.75 + 0.5 * LA) / B.alpha * s0, eb = (0.75 + 0.5 * LB) / B.beta * s0;
    double* g = A.part + (int64_t)(blockIdx.x % (unsigned)A.n_slices) * A.slice_stride;
    for (int x = 0; x < 3; ++x) {
        const int ix = x == 0, iy = x == 1, iz = x == 2;
        double ga = ta * at(a[0] + ix, a[1] + iy, a[2] + iz, b[0], b[1], b[2]);
        double gb = tb * at(a[0], a[1], a[2], b[0] + ix, b[1] + iy, b[2] + iz);
        if (a[x]) ga = fma((double)-a[x], at(a[0] - ix, a[1] - iy, a[2] - iz, b[0], b[1], b[2]), ga);
        if (b[x]) gb = fma((double)-b[x], at(a[0], a[1], a[2], b[0] - ix, b[1] - iy, b[2] - iz), gb);
        unsafeAtomicAdd(g + 3 * (int64_t)S.sa + x, d * ga);
        unsafeAtomicAdd(g + 3 * (int64_t)S.sb + x, d * gb);
        ea -= at(a[0] + 2 * ix, a[1] + 2 * iy, a[2] + 2 * iz, b[0], b[1], b[2]);
        eb -= at(a[0], a[1], a[2], b[0] + 2 * ix, b[1] + 2 * iy, b[2] + 2 * iz);
    }
    const int k = (int)(A.prim0 + i - S.prim_off);
    unsafeAtomicAdd(g + A.ns3 + A.poff[S.sa] + k / S.kb, d * ea);
    unsafeAtomicAdd(g + A.ns3 + A.poff[S.sb] + k % S.kb, d * eb);
}

__global__ __launch_bounds__(256) void coul_zero_kernel(double* __restrict__ x, int64_t n)
{
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)gridDim.x * 256) x[t] = 0.0;
}

// grad_c / grad_e += the sum of the slices, in slice order.
__global__ __launch_bounds__(256) void coul_reduce_kernel(const double* __restrict__ part, int n_slices, int64_t n_grad,
                                                          int64_t ns3, double* __restrict__ grad_c,
                                                          double* __restrict__ grad_e)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n_grad) return;
    double v = 0.0;
    for (int b = 0; b < n_slices; ++b) v += part[(int64_t)b * n_grad + t];
    if (t < ns3)
        grad_c[t] += v;
    else
        grad_e[t - ns3] += v;
}

// energy[0] += the sum of the jobs' shares, in a fixed order with two-sum
// compensation (one workgroup).
__global__ __launch_bounds__(1024) void coul_energy_kernel(const double* __restrict__ x, int64_t n,
                                                           double* __restrict__ energy)
{
    __shared__ double s_hi[1024], s_lo[1024];
    double hi = 0.0, lo = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) {
        eri_coul_add(hi, lo, x[2 * i]);
        lo += x[2 * i + 1];
    }
    s_hi[threadIdx.x] = hi;
    s_lo[threadIdx.x] = lo;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            double s, e;
            eri_two_sum(s_hi[threadIdx.x], s_hi[threadIdx.x + w], s, e);
            s_hi[threadIdx.x] = s;
            s_lo[threadIdx.x] = s_lo[threadIdx.x] + s_lo[threadIdx.x + w] + e;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) energy[0] += s_hi[0] + s_lo[0];
}

const void* const CHARGE[NCLS] = {(const void*)coul_charge_kernel<0, 0>, (const void*)coul_charge_kernel<1, 0>,
                                  (const void*)coul_charge_kernel<1, 1>, (const void*)coul_charge_kernel<2, 0>,
                                  (const void*)coul_charge_kernel<2, 1>, (const void*)coul_charge_kernel<2, 2>};
const void* const GRADIENT[NCLS] = {(const void*)coul_gradient_kernel<0, 0>, (const void*)coul_gradient_kernel<1, 0>,
                                    (const void*)coul_gradient_kernel<1, 1>, (const void*)coul_gradient_kernel<2, 0>,
                                    (const void*)coul_gradient_kernel<2, 1>, (const void*)coul_gradient_kernel<2, 2>};

// Fewest sources of a job: some 12000 of the step's fma (R's recursion, and R
// into V) and 150 for the Boys function, so that what a wavefront does once
// (its table columns, its targets, its additions into V: 20 us) stays small
// beside its walk, and one job's walk stays short beside a launch.  One size
// of 64 for all kernels left the 49 jobs of (dd|dd) in a 24-atom basis
// running alone for 0.9 ms.
int chunk_min(int lt, int ls)
{
    const int n = lt + ls + 2;
    const int step = (n + 1) * (n + 2) * (n + 3) * (n + 4) / 24 + nherm(lt + 2) * nherm(ls) + 150;
    return std::min(64, std::max(8, 12000 / step));
}

// The targets of one half of a batch entry: shell pairs [tp0, tp0 + lo.size())
// with the source shell pairs [lo[k], hi[k]).
struct half_entry {
    int tc, sc;
    int64_t tp0;
    std::vector<int32_t> lo, hi;
};

// Both halves of a batch entry.  The entry lists, for each bra pair in
// decreasing order of Q, a prefix of the ket pairs (also in decreasing order),
// so the bra pairs of one ket pair are a range too: up to the last one whose
// prefix reaches it, from the first, or, where bra and ket are one group
// (prefixes cut at the bra pair itself), from the ket pair on.
void split_entry(const eri_plan* p, const eri_batch_class& bc, std::vector<half_entry>& out)
{
    const int tc = cls_of(bc.cid >> 6, (bc.cid >> 4) & 3), sc = cls_of((bc.cid >> 2) & 3, bc.cid & 3);
    half_entry f{tc, sc, p->h_seg_p1[bc.seg_lo], {}, {}}, t{sc, tc, bc.ket_lo, {}, {}};
    const bool one_group = f.tp0 == bc.ket_lo;
    int64_t reach = 0;
    for (int64_t s = bc.seg_lo; s < bc.seg_hi; ++s) {
        const int64_t n = p->h_seg_off[s + 1] - p->h_seg_off[s];
        f.lo.push_back((int32_t)bc.ket_lo);
        f.hi.push_back((int32_t)(bc.ket_lo + n));
        reach = std::max(reach, n);
    }
    t.lo.assign(reach, 0);
    t.hi.assign(reach, 0);
    int64_t done = 0;
    for (int64_t s = bc.seg_hi - 1; s >= bc.seg_lo; --s) {
        const int64_t n = p->h_seg_off[s + 1] - p->h_seg_off[s];
        for (; done < n; ++done) {
            t.lo[done] = one_group ? (int32_t)(bc.ket_lo + done + 1) : p->h_seg_p1[bc.seg_lo];
            t.hi[done] = p->h_seg_p1[s] + 1;
        }
    }
    out.push_back(std::move(f));
    out.push_back(std::move(t));
}

int build(eri_plan* p, eri_coul_state* st)
{
    const int64_t np = (int64_t)p->h_pairs.size(), ns = (int64_t)p->sh_L.size();
    auto prim_at = [&](int64_t pair) { return pair < np ? p->h_pairs[pair].prim_off : p->n_prims; };
    std::vector<int32_t> prim_pair(p->n_prims);
    int64_t first[NCLS + 1];
    std::fill(first, first + NCLS + 1, np);
    for (int64_t i = np - 1; i >= 0; --i) {
        const eri_shell_pair& s = p->h_pairs[i];
        first[cls_of(p->sh_L[s.sa], p->sh_L[s.sb])] = i;
        for (int k = 0; k < s.nprim; ++k) prim_pair[s.prim_off + k] = (int32_t)i;
    }
    for (int c = NCLS - 1; c >= 0; --c) first[c] = std::min(first[c], first[c + 1]);   // a class without pairs
    for (int c = 0; c <= NCLS; ++c) st->prim0[c] = prim_at(first[c]);
    for (int c = 0; c < NCLS; ++c) {
        const int64_t n = st->prim0[c + 1] - st->prim0[c];
        const int L = CLS_LA[c] + CLS_LB[c];
        st->rec0[c] = st->n_rec;
        st->n_rec += n * (4 + nherm(L));
        st->pot0[c] = st->n_pot;
        st->n_pot += n * nherm(L + 2);
    }
    // ---- ranges, and the wavefronts' source ranges -------------------------------
    std::vector<half_entry> halves;
    for (const auto& bc : p->bclass) split_entry(p, bc, halves);
    std::vector<eri_coul_range> ranges;
    std::vector<eri_coul_job> whole;      // one per block of 64 targets and half entry
    std::vector<int> kern;
    int64_t total[25] = {};               // source steps of each kernel
    for (const half_entry& h : halves) {
        const int64_t base = (int64_t)ranges.size() - h.tp0;
        for (size_t k = 0; k < h.lo.size(); ++k) {
            eri_coul_range r{(int32_t)prim_at(h.lo[k]), (int32_t)prim_at(h.hi[k])};
            if (h.hi[k] <= h.lo[k]) r.hi = r.lo;
            ranges.push_back(r);
        }
        const int64_t t1 = prim_at(h.tp0 + (int64_t)h.lo.size());
        const int LT = CLS_LA[h.tc] + CLS_LB[h.tc], LS = CLS_LA[h.sc] + CLS_LB[h.sc];
        for (int64_t t0 = prim_at(h.tp0); t0 < t1; t0 += 64) {
            eri_coul_job j;
            j.t0 = (int32_t)t0;
            j.n = (int32_t)std::min<int64_t>(64, t1 - t0);
            j.lo = INT32_MAX;
            j.hi = 0;
            for (int64_t q = prim_pair[t0]; q <= prim_pair[t0 + j.n - 1]; ++q) {
                const eri_coul_range& r = ranges[base + q];
                if (r.hi <= r.lo) continue;
                j.lo = std::min(j.lo, r.lo);
                j.hi = std::max(j.hi, r.hi);
            }
            if (j.hi <= j.lo) continue;
            j.s0 = (int32_t)st->prim0[h.sc];
            j.trec = st->rec0[h.tc] + (t0 - st->prim0[h.tc]) * (4 + nherm(LT));
            j.srec = st->rec0[h.sc];
            j.tpot = st->pot0[h.tc] + (t0 - st->prim0[h.tc]);
            j.pot_stride = (int32_t)(st->prim0[h.tc + 1] - st->prim0[h.tc]);
            j.range = base;
            total[5 * LT + LS] += j.hi - j.lo;
            whole.push_back(j);
            kern.push_back(5 * LT + LS);
        }
    }
    // ---- jobs: the ranges in pieces, so that there are enough of them ------------
    std::vector<eri_coul_job> jobs;
    for (int k = 0; k < 25; ++k) {
        st->job0[k] = (int64_t)jobs.size();
        const int chunk = (int)std::min<int64_t>(COUL_CHUNK_MAX, std::max<int64_t>(chunk_min(k / 5, k % 5), total[k] / COUL_JOBS));
        for (size_t w = 0; w < whole.size(); ++w) {
            if (kern[w] != k) continue;
            eri_coul_job j = whole[w];
            const int hi = j.hi;
            for (; j.lo < hi; j.lo = j.hi) {
                j.hi = std::min(hi, j.lo + chunk);
                jobs.push_back(j);
            }
        }
    }
    st->job0[25] = (int64_t)jobs.size();
    if (jobs.size() > (size_t)INT32_MAX) return ERI_EUNSUPPORTED;
    std::vector<int64_t> bf(ns + 1, 0);
    for (int64_t s = 0; s < ns; ++s) bf[s + 1] = bf[s] + ncart(p->sh_L[s]);
    st->nbf = bf[ns];
    st->n_grad = 3 * ns + (int64_t)p->sh_exps.size();
    st->n_slices = (int)std::max<int64_t>(1, std::min<int64_t>(COUL_SLICES_MAX, COUL_SLICE_DOUBLES / std::max<int64_t>(1, st->n_grad)));
    ERI_TRY(upload(p, (void**)&st->d_jobs, jobs.empty() ? nullptr : jobs.data(), jobs.size() * sizeof(eri_coul_job)));
    ERI_TRY(upload(p, (void**)&st->d_ranges, ranges.empty() ? nullptr : ranges.data(), ranges.size() * sizeof(eri_coul_range)));
    ERI_TRY(upload(p, (void**)&st->d_prim_pair, prim_pair.empty() ? nullptr : prim_pair.data(), prim_pair.size() * sizeof(int32_t)));
    ERI_TRY(upload(p, (void**)&st->d_bf, bf.data(), bf.size() * sizeof(int64_t)));
    ERI_TRY(upload(p, (void**)&st->d_poff, p->sh_off.empty() ? nullptr : p->sh_off.data(), p->sh_off.size() * sizeof(int64_t)));
    ERI_TRY(upload(p, (void**)&st->d_rec, nullptr, 2 * (size_t)st->n_rec * sizeof(double)));
    ERI_TRY(upload(p, (void**)&st->d_pot, nullptr, (size_t)st->n_pot * sizeof(double)));
    ERI_TRY(upload(p, (void**)&st->d_energy, nullptr, 2 * jobs.size() * sizeof(double)));
    ERI_TRY(upload(p, (void**)&st->d_part, nullptr, (size_t)st->n_slices * st->n_grad * sizeof(double)));
    return ERI_OK;
}

int launch(const void* fn, int64_t grid, int rows, int block, void* args, hipStream_t strm)
{
    if (grid <= 0) return ERI_OK;
    void* a[] = {args};
    ERI_HIP_TRY(hipLaunchKernel(fn, dim3((unsigned)grid, (unsigned)rows), dim3(block), a, 0, strm));
    return ERI_OK;
}

}  // namespace

int eri_grad_zero(double* x, int64_t n, hipStream_t strm)
{
    if (n <= 0) return ERI_OK;
    const unsigned g = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(coul_zero_kernel, dim3(g), dim3(256), 0, strm, x, n);
    ERI_HIP_TRY(hipGetLastError());
    return ERI_OK;
}

int eri_grad_reduce(const double* part, int n_slices, int64_t n_grad, int64_t ns3, double* grad_c, double* grad_e,
                    hipStream_t strm)
{
    if (n_grad <= 0) return ERI_OK;
    hipLaunchKernelGGL(coul_reduce_kernel, dim3((unsigned)((n_grad + 255) / 256)), dim3(256), 0, strm, part, n_slices,
                       n_grad, ns3, grad_c, grad_e);
    ERI_HIP_TRY(hipGetLastError());
    return ERI_OK;
}

int eri_energy_add(const double* shares, int64_t n, double* energy, hipStream_t strm)
{
    hipLaunchKernelGGL(coul_energy_kernel, dim3(1), dim3(1024), 0, strm, shares, n, energy);
    ERI_HIP_TRY(hipGetLastError());
    return ERI_OK;
}

int eri_coul_backward(eri_plan* p, hipStream_t strm, const double* density, int64_t nbf, double* grad_c, double* grad_e,
                      double* energy)
{
    if (!p->coul) {
        eri_coul_state* st = new (std::nothrow) eri_coul_state();
        if (!st) return ERI_ENOMEM;
        int rc;
        try {
            rc = build(p, st);
        } catch (const std::bad_alloc&) {
            rc = ERI_ENOMEM;
        }
        if (rc != ERI_OK) {
            eri_coul_free(st);
            return rc;
        }
        p->coul = st;
    }
    eri_coul_state* st = p->coul;
    if (nbf != st->nbf) return ERI_EINVAL;
    coul_pair_args a;
    std::memset(&a, 0, sizeof(a));
    a.pairs = p->d_pairs;
    a.prims = p->d_prims;
    a.prim_pair = st->d_prim_pair;
    a.bf = st->d_bf;
    a.poff = st->d_poff;
    a.dens = density;
    a.nbf = nbf;
    a.part = st->d_part;
    a.slice_stride = st->n_grad;
    a.ns3 = 3 * (int64_t)p->sh_L.size();
    a.n_slices = st->n_slices;
    auto per_class = [&](const void* const* fn, bool components) {
        for (int c = 0; c < NCLS; ++c) {
            a.prim0 = st->prim0[c];
            a.n = st->prim0[c + 1] - st->prim0[c];
            a.full = st->d_rec + st->rec0[c];
            a.rec = a.full + st->n_rec;
            a.pot = st->d_pot + st->pot0[c];
            a.pot_stride = a.n;
            ERI_TRY(launch(fn[c], (a.n + 63) / 64, components ? ncart(CLS_LA[c]) * ncart(CLS_LB[c]) : 1, 64, &a, strm));
        }
        return (int)ERI_OK;
    };
    ERI_TRY(per_class(CHARGE, false));
    if (grad_c) ERI_TRY(eri_grad_zero(st->d_pot, st->n_pot, strm));
    for (int k = 24; k >= 0; --k) {   // the longest first
        eri_coul_args c;
        c.jobs = st->d_jobs + st->job0[k];
        c.n_jobs = st->job0[k + 1] - st->job0[k];
        c.full = st->d_rec;
        c.rec = st->d_rec + st->n_rec;
        c.ranges = st->d_ranges;
        c.prim_pair = st->d_prim_pair;
        c.pot = st->d_pot;
        c.energy = st->d_energy + 2 * st->job0[k];
        ERI_TRY(launch(eri_coul_kernel(k / 5, k % 5, grad_c != nullptr), (c.n_jobs + 3) / 4, 1, 256, &c, strm));
    }
    if (grad_c) {
        ERI_TRY(eri_grad_zero(st->d_part, (int64_t)st->n_slices * st->n_grad, strm));
        ERI_TRY(per_class(GRADIENT, true));
        ERI_TRY(eri_grad_reduce(st->d_part, st->n_slices, st->n_grad, a.ns3, grad_c, grad_e, strm));
    }
    if (energy) ERI_TRY(eri_energy_add(st->d_energy, st->job0[25], energy, strm));
    return ERI_OK;
}
