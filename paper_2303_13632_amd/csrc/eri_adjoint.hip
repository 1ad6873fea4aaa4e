// The adjoint of a short explicit list: a workgroup per quartet, side and
// a few of its primitive pairs, every class in one launch.
//
// With Gbar general (no product of densities), L of one quartet is
//   sum_ij sum_t,t' [sum_x,y E_i[x][t] Gbar[x][y] E_j[y][t']] R_(t+t')
// over its primitive pairs i, j (x, y: component pairs of bra and ket, E their
// Hermite expansions, R the Hermite Coulomb integrals; McMurchie and Davidson's
// scheme).  For each side as target, batches of source primitive pairs j are
// contracted with Gbar first,
//   g_j[x][t'] = sum_y Gbar[x][y] E_j[y][t'],
// then for every target primitive pair i
//   U[x][t] = sum_j sum_t' g_j[x][t'] R_(t+t'),  |t| <= La + Lb + 2,
// whose products with the expansions of the differentiated Gaussians (a + 1, a - 1
// and a + 2 at either centre) are the quartet's gradient.  Both sides are
// targets, so all four centres are differentiated explicitly.
//
// Why such small pieces and all sizes at run time: a list of a few
// hundred quartets spreads over up to 81 classes.  The derived-class path
// (eri_backward.hip) launches some 30 kernels per class and waits for the
// stream once per class and exponent; 256 quartets of s, p, d shells took
// 29.5 ms there (values and gradient), 0.9 ms here.  That path shares the recurrences of a class over
// many quartets and wins on classes of many or deep ones (eri_adj_routes).
// Bound by the serial chain of a workgroup (levels of R, LDS round trips).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "eri_coulomb.h"
#include "eri_internal.h"

using namespace eri_detail;

namespace {

constexpr int ADJ_IB = 8;           // target primitive pairs whose Boys values are staged together
constexpr int64_t ADJ_WORK = 4096;  // workgroups aimed at (16 a CU)
constexpr int ADJ_SLICES_MAX = 64;
constexpr int64_t ADJ_SLICE_DOUBLES = (int64_t)1 << 22;   // gradient slices in all (32 MB; they span every shell of the plan)

// One class of the list.
struct adj_class {
    int64_t first;      // first item
    int64_t eoff;       // first ERI
    int32_t L[4];       // user shells
    int32_t jc;         // source primitive pairs per batch
    int32_t pad;
};

// One workgroup's work: target primitive pairs [i0, i0 + in) of one side of an item.
struct adj_work {
    int32_t item, cls;
    int16_t side, i0, in, pad;
    int32_t share;      // place of its share of L, or -1 (side 1; classes whose L comes from elsewhere)
};

struct adj_args {
    const eri_item* items;          // user order: bra = record of (a, b), ket = record of (c, d); sign bit: the
                                    // record holds the two shells in the other order
    const eri_shell_pair* pairs;
    const eri_prim_pair* prims;
    const adj_class* cls;
    const adj_work* work;
    int grad;                       // 0: L alone
    const double* dl;               // Gbar, or null:
    const double* dens;
    const int64_t* bf;
    int64_t nbf;
    const int64_t* poff;
    double* part;
    int64_t slice_stride, ns3;
    int n_slices;
    double* energy;                 // shares of L (value, 0)
};

__host__ __device__ constexpr int adj_nherm(int L) { return (L + 1) * (L + 2) * (L + 3) / 6; }
__host__ __device__ constexpr int adj_nc(int L) { return (L + 1) * (L + 2) / 2; }
__host__ __device__ constexpr int adj_pad4(int n) { return (n + 3) & ~3; }

// Doubles of LDS of a class, the same formulas on the host and in the kernel.
struct adj_lds {
    int h, off, cx, G, Ey, EE, g, base, lev, R, Ex, end;
    // bra and ket orders, components and the batch size; each buffer holds
    // what either side as target needs
    __host__ __device__ adj_lds(const int L[4], int jc)
    {
        const int lb = L[0] + L[1], lk = L[2] + L[3], N = lb + lk + 2;
        const int nb = adj_nc(L[0]) * adj_nc(L[1]), nk = adj_nc(L[2]) * adj_nc(L[3]);
        const int hb = adj_nherm(lb), hk = adj_nherm(lk);
        const int lm = lb > lk ? lb : lk;
        auto mx = [](int a, int b) { return a > b ? a : b; };
        int o = 0;
        h = o;      o += (adj_nherm(N) + 1) / 2;                                   // packed (t, u, v) as int
        off = o;    o += (adj_pad4(adj_nherm(lm)) + 1) / 2;                        // place of t' in the cube
        cx = o;     o += (adj_pad4(mx(nb, nk)) + 1) / 2;                           // components of x, packed
        G = o;      o += mx(nb * adj_pad4(nk), nk * adj_pad4(nb));                  // [y][x]
        g = adj_pad4(o); o = g + jc * mx(adj_pad4(hk) * adj_pad4(nb), adj_pad4(hb) * adj_pad4(nk));   // [j][t'][x]
        Ey = o;     o += jc * 27 * (lm + 1);                                       // [j][axis][c][d][t]
        // EE and what replaces it once g is formed
        EE = o;
        int p = EE;
        base = p;   p += ADJ_IB * jc * (N + 4);                                    // F and P - Q of (i, j)
        lev = p;    p += 3 * jc * level_max(N);
        R = p;      p += jc * (N + 1) * (N + 1) * (N + 1);
        Ex = p;     p += 75 * (lm + 3);
        o = EE + mx(p - EE, jc * mx(nk * hk, nb * hb));
        end = o;
    }
    // most values (t, u, v; m) of one level of R's recursion
    __host__ __device__ static int level_max(int N)
    {
        int m = 0;
        for (int n = 0; n <= N; ++n) m = m > adj_nc(n) * (N - n + 1) ? m : adj_nc(n) * (N - n + 1);
        return m;
    }
};

// E[t], t <= 6, of x_A^a x_B^b about P (one axis), zero beyond a + b.
__device__ __forceinline__ void adj_hermite(int a, int b, double h, double pa, double pb, double (&e)[7])
{
    e[0] = 1.0;
#pragma unroll
    for (int t = 1; t < 7; ++t) e[t] = 0.0;
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        if (s >= a + b) break;
        const double x = s < a ? pa : pb;
        double n[7];
#pragma unroll
        for (int t = 0; t < 7; ++t) {
            double v = x * e[t];
            if (t > 0) v = fma(h, e[t - 1], v);
            if (t < 6) v = fma((double)(t + 1), e[t + 1], v);
            n[t] = v;
        }
#pragma unroll
        for (int t = 0; t < 7; ++t) e[t] = n[t];
    }
}

// Exponents of component idx of a Cartesian shell (x^L first), one byte each.
__device__ __forceinline__ int adj_comp(int L, int idx)
{
    int m = 0;
    while ((m + 1) * (m + 2) / 2 <= idx) ++m;
    const int z = idx - m * (m + 1) / 2;
    return (L - m) | (m - z) << 8 | z << 16;
}

__device__ __forceinline__ double adj_wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

template <int NT>
__global__ __launch_bounds__(NT) void adj_list_kernel(adj_args A)
{
    extern __shared__ __align__(32) double s[];
    __shared__ double s_gc[2][3], s_ge[2][ERI_MAX_K], s_red[NT];
    const int tid = threadIdx.x;
    const adj_work W = A.work[blockIdx.x];
    const adj_class& C = A.cls[W.cls];
    const int64_t idx = W.item - C.first;
    const eri_item it = A.items[W.item];
    int L[4] = {C.L[0], C.L[1], C.L[2], C.L[3]};
    const int jc = C.jc;
    const adj_lds Z(L, jc);
    int* s_h = reinterpret_cast<int*>(s + Z.h);
    double* s_G = s + Z.G;
    // records of the two pairs; rev: the record holds (b, a) of the user's (a, b)
    const eri_shell_pair P[2] = {A.pairs[it.bra & 0x7fffffff], A.pairs[it.ket & 0x7fffffff]};
    const bool rev[2] = {it.bra < 0, it.ket < 0};
    const int LA[2] = {rev[0] ? L[1] : L[0], rev[1] ? L[3] : L[2]};
    const int LB[2] = {rev[0] ? L[0] : L[1], rev[1] ? L[2] : L[3]};
    const int nA[2] = {adj_nc(LA[0]), adj_nc(LA[1])}, nB[2] = {adj_nc(LB[0]), adj_nc(LB[1])};
    const int nx[2] = {nA[0] * nB[0], nA[1] * nB[1]}, Lp[2] = {LA[0] + LB[0], LA[1] + LB[1]};
    const int N = Lp[0] + Lp[1] + 2;
    for (int i = tid; i < adj_nherm(N); i += NT) {
        int n = 0;
        while (adj_nherm(n) <= i) ++n;
        const int k = i - (n ? adj_nherm(n - 1) : 0);
        int m = 0;
        while ((m + 1) * (m + 2) / 2 <= k) ++m;
        const int v = k - m * (m + 1) / 2;
        s_h[i] = (n - m) | (m - v) << 8 | v << 16;
    }
    if (tid < 6) s_gc[tid / 3][tid % 3] = 0.0;
    if (tid < 2 * ERI_MAX_K) s_ge[tid / ERI_MAX_K][tid % ERI_MAX_K] = 0.0;
    // ---- Gbar in record order, [y][x]: target components on consecutive lanes ----
    {
        const int st3 = 1, st2 = adj_nc(L[3]), st1 = st2 * adj_nc(L[2]), st0 = st1 * adj_nc(L[1]);
        const int ba = rev[0] ? st1 : st0, bb = rev[0] ? st0 : st1, ka = rev[1] ? st3 : st2, kb = rev[1] ? st2 : st3;
        const double* row = A.dl ? A.dl + C.eoff + idx * (int64_t)(nx[0] * nx[1]) : nullptr;
        const int nXp = adj_pad4(nx[W.side]);
        for (int k = tid; k < nx[0] * nx[1]; k += NT) {
            const int x = k / nx[1], y = k - x * nx[1];
            const int i0 = x / nB[0], i1 = x - i0 * nB[0], i2 = y / nB[1], i3 = y - i2 * nB[1];
            s_G[W.side == 0 ? y * nXp + x : x * nXp + y] = row ? row[i0 * ba + i1 * bb + i2 * ka + i3 * kb]
                         // the density's element in the user's order of the pair
                         : (rev[0] ? A.dens[(A.bf[P[0].sb] + i1) * A.nbf + A.bf[P[0].sa] + i0]
                                   : A.dens[(A.bf[P[0].sa] + i0) * A.nbf + A.bf[P[0].sb] + i1]) *
                               (rev[1] ? A.dens[(A.bf[P[1].sb] + i3) * A.nbf + A.bf[P[1].sa] + i2]
                                       : A.dens[(A.bf[P[1].sa] + i2) * A.nbf + A.bf[P[1].sb] + i3]);
        }
    }
    double energy = 0.0;
    {
        const int side = W.side;
        const int o = side ^ 1;
        const eri_shell_pair X = P[side], Y = P[o];
        const int LX = Lp[side], LY = Lp[o], la = LA[side], lb = LB[side], lc = LA[o], ld = LB[o];
        const int nX = nx[side], nY = nx[o], nXp = adj_pad4(nX), ht = adj_nherm(LX + 2), hs = adj_nherm(LY);
        const int cube = (N + 1) * (N + 1) * (N + 1), lmax = adj_lds::level_max(N);
        const int dE = (la + 3) * (lb + 3) * (LX + 3);
        const int hsp = adj_pad4(hs), bs = N + 4;
        int* s_off = reinterpret_cast<int*>(s + Z.off);
        int* s_cx = reinterpret_cast<int*>(s + Z.cx);
        __syncthreads();   // s_h
        for (int k = tid; k < hsp; k += NT) {
            const int q = k < hs ? s_h[k] : 0;
            s_off[k] = ((q & 255) * (N + 1) + ((q >> 8) & 255)) * (N + 1) + (q >> 16);
        }
        for (int k = tid; k < nX; k += NT) s_cx[k] = adj_comp(la, k / nB[side]) | adj_comp(lb, k % nB[side]) << 4;
        double cA[3] = {0.0, 0.0, 0.0}, cB[3] = {0.0, 0.0, 0.0};
        for (int jb = 0; jb < Y.nprim; jb += jc) {
            const int jn = min(jc, Y.nprim - jb);
            __syncthreads();   // the buffers of the batch before are read
            // expansions of the batch's source pairs: (j, axis, c, d)
            const int ncd = (lc + 1) * (ld + 1);
            for (int k = tid; k < jn * 3 * ncd; k += NT) {
                const int j = k / (3 * ncd), r = k - j * 3 * ncd, ax = r / ncd, cd = r - ax * ncd;
                const eri_prim_pair Q = A.prims[Y.prim_off + jb + j];
                const double pa = ax == 0 ? Q.PA[0] : ax == 1 ? Q.PA[1] : Q.PA[2];
                const double ab = ax == 0 ? Y.AB[0] : ax == 1 ? Y.AB[1] : Y.AB[2];
                double e[7];
                adj_hermite(cd / (ld + 1), cd % (ld + 1), Q.hp, pa, Q.alpha / Q.p * ab, e);
#pragma unroll
                for (int t = 0; t < 7; ++t)
                    if (t <= LY) s[Z.Ey + k * (LY + 1) + t] = e[t];
            }
            __syncthreads();
            // E_j[y][t'] with the pair's prefactor and (-1)^|t'|
            for (int k = tid; k < jn * nY * hs; k += NT) {
                const int j = k / (nY * hs), r = k - j * nY * hs, y = r / hs, h = s_h[r - y * hs];
                const int a = adj_comp(lc, y / nB[o]), b = adj_comp(ld, y % nB[o]);
                double v = A.prims[Y.prim_off + jb + j].kp;
                for (int ax = 0; ax < 3; ++ax) {
                    const int t = (h >> 8 * ax) & 255, ca = (a >> 8 * ax) & 255, cb = (b >> 8 * ax) & 255;
                    v *= s[Z.Ey + (((j * 3 + ax) * (lc + 1) + ca) * (ld + 1) + cb) * (LY + 1) + t];
                    if (t & 1) v = -v;
                }
                s[Z.EE + k] = v;
            }
            __syncthreads();
            // g_j[t'][x] = sum_y Gbar[x][y] E_j[y][t']
            for (int k = tid; k < jn * hsp * nXp; k += NT) {
                const int j = k / (hsp * nXp), r = k - j * hsp * nXp, t = r / nXp, x = r - t * nXp;
                double v = 0.0;
                if (x < nX && t < hs) {
                    const double* e = s + Z.EE + j * nY * hs + t;
#pragma unroll 6
                    for (int y = 0; y < nY; ++y) v = fma(s_G[y * nXp + x], e[y * hs], v);
                }
                s[Z.g + k] = v;
            }
            const int iend = W.i0 + W.in;
            for (int ib = W.i0; ib < iend; ib += ADJ_IB) {
                const int in = min(ADJ_IB, iend - ib);
                __syncthreads();   // EE is read; the block before is done
                // R^m_000 of the block's (i, j)
                for (int k = tid; k < in * jn; k += NT) {
                    const eri_prim_pair B = A.prims[X.prim_off + ib + k / jn], Q = A.prims[Y.prim_off + jb + k % jn];
                    const double ir = eri_coul_rsqrt(B.p + Q.p), rho = B.p * Q.p * ir * ir;
                    const double x = B.P[0] - Q.P[0], y = B.P[1] - Q.P[1], z = B.P[2] - Q.P[2];
                    double F[11];   // orders above N are computed and dropped
                    eri_boys<10>(rho * fma(x, x, fma(y, y, z * z)), F);
                    double f = ERI_TWO_PI_52 * ir * B.kp;
#pragma unroll
                    for (int m = 0; m < 11; ++m) {
                        if (m <= N) s[Z.base + k * bs + m] = f * F[m];
                        f *= -2.0 * rho;
                    }
                    s[Z.base + k * bs + N + 1] = x;
                    s[Z.base + k * bs + N + 2] = y;
                    s[Z.base + k * bs + N + 3] = z;
                }
                for (int i = 0; i < in; ++i) {
                    const eri_prim_pair B = A.prims[X.prim_off + ib + i];
                    __syncthreads();   // the target before is done; the base values are there
                    // expansions of the target: (axis, a, b), a <= la + 2, b <= lb + 2
                    for (int k = tid; k < 3 * (la + 3) * (lb + 3); k += NT) {
                        const int ax = k / ((la + 3) * (lb + 3)), r = k - ax * (la + 3) * (lb + 3);
                        const int a = r / (lb + 3), b = r - a * (lb + 3);
                        const double pa = ax == 0 ? B.PA[0] : ax == 1 ? B.PA[1] : B.PA[2];
                        const double ab = ax == 0 ? X.AB[0] : ax == 1 ? X.AB[1] : X.AB[2];
                        double e[7];
                        adj_hermite(a, b, B.hp, pa, B.alpha / B.p * ab, e);
#pragma unroll
                        for (int t = 0; t < 7; ++t)
                            if (t <= LX + 2) s[Z.Ex + k * (LX + 3) + t] = a + b <= LX + 2 ? e[t] : 0.0;
                    }
                    // R of the batch, level by level; level n holds [j][k][m], m <= N - n
                    for (int n = 0; n <= N; ++n) {
                        const int nm = N - n + 1, nk = adj_nc(n), hb = n ? adj_nherm(n - 1) : 0;
                        double* cur = s + Z.lev + (n % 3) * jc * lmax;
                        const double* p1 = s + Z.lev + ((n + 2) % 3) * jc * lmax;
                        const double* p2 = s + Z.lev + ((n + 1) % 3) * jc * lmax;
                        // r / nm as a product: exact for the r < 4 * 144 here
                        const int a1 = nk * nm, magic = 65536 / nm + 1;
                        for (int k = tid; k < jn * a1; k += NT) {
                            const int j = (k >= a1) + (k >= 2 * a1) + (k >= 3 * a1);
                            const int r = k - j * a1, q = (r * magic) >> 16, m = r - q * nm;
                            double v;
                            int h = 0;
                            if (n == 0) {
                                v = s[Z.base + (i * jn + j) * bs + m];
                            } else {
                                h = s_h[hb + q];
                                const int t = h & 255, u = (h >> 8) & 255, w = h >> 16;
                                const int ax = t ? 0 : u ? 1 : 2, low = (t ? t : u ? u : w) - 1;
                                const double d = s[Z.base + (i * jn + j) * bs + N + 1 + ax];
                                // (t, u, v) lowered: its place within the level below
                                const int u1 = u - (ax == 1), w1 = w - (ax == 2), m1 = u1 + w1;
                                const int q1 = m1 * (m1 + 1) / 2 + w1;
                                v = d * p1[(j * adj_nc(n - 1) + q1) * (nm + 1) + m + 1];
                                if (low) {
                                    const int u2 = u1 - (ax == 1), w2 = w1 - (ax == 2), m2 = u2 + w2;
                                    const int q2 = m2 * (m2 + 1) / 2 + w2;
                                    v = fma((double)low, p2[(j * adj_nc(n - 2) + q2) * (nm + 2) + m + 1], v);
                                }
                            }
                            cur[(j * nk + q) * nm + m] = v;
                            if (m == 0)
                                s[Z.R + j * cube + ((h & 255) * (N + 1) + ((h >> 8) & 255)) * (N + 1) + (h >> 16)] = v;
                        }
                        __syncthreads();
                    }
                    // U[x][t] of four x at a time, and its share of every derivative
                    double ea = 0.0, eb = 0.0;
                    const double ta = 2.0 * B.alpha, tb = 2.0 * B.beta;
                    const double na = (0.75 + 0.5 * la) / B.alpha, nb = (0.75 + 0.5 * lb) / B.beta;
                    for (int k = tid; k < (nXp / 4) * ht; k += NT) {
                        const int xg = k / ht, h = s_h[k - xg * ht];
                        const int tx = h & 255, ty = (h >> 8) & 255, tz = h >> 16;
                        const double* Rt = s + Z.R + (tx * (N + 1) + ty) * (N + 1) + tz;
                        double U[4] = {0.0, 0.0, 0.0, 0.0};
                        for (int j = 0; j < jn; ++j) {
                            const double* g = s + Z.g + j * hsp * nXp + 4 * xg;
                            for (int t = 0; t < hsp; t += 4, g += 4 * nXp)
#pragma unroll
                                for (int w = 0; w < 4; ++w) {
                                    const double r = Rt[j * cube + s_off[t + w]];
#pragma unroll
                                    for (int e = 0; e < 4; ++e) U[e] = fma(g[w * nXp + e], r, U[e]);
                                }
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int x = 4 * xg + e;
                            if (x >= nX) continue;
                            const int c = s_cx[x];
                            const double* E[3];
                            double e0[3];
                            const int sa = (lb + 3) * (LX + 3), sb = LX + 3;
#pragma unroll
                            for (int ax = 0; ax < 3; ++ax) {
                                const int a = (c >> 8 * ax) & 15, b = (c >> (8 * ax + 4)) & 15;
                                E[ax] = s + Z.Ex + ax * dE + a * sa + b * sb + (ax == 0 ? tx : ax == 1 ? ty : tz);
                                e0[ax] = E[ax][0];
                            }
                            const double whole = e0[0] * e0[1] * e0[2];
                            energy += side == 0 ? U[e] * whole : 0.0;
                            double da = na * whole, db = nb * whole;
#pragma unroll
                            for (int ax = 0; ax < 3; ++ax) {
                                const int a = (c >> 8 * ax) & 15, b = (c >> (8 * ax + 4)) & 15;
                                const double w = ax == 0 ? e0[1] * e0[2] : ax == 1 ? e0[0] * e0[2] : e0[0] * e0[1];
                                double ga = ta * E[ax][sa], gb = tb * E[ax][sb];
                                if (a) ga = fma((double)-a, E[ax][-sa], ga);
                                if (b) gb = fma((double)-b, E[ax][-sb], gb);
                                cA[ax] = fma(U[e] * w, ga, cA[ax]);
                                cB[ax] = fma(U[e] * w, gb, cB[ax]);
                                da = fma(-w, E[ax][2 * sa], da);
                                db = fma(-w, E[ax][2 * sb], db);
                            }
                            ea = fma(U[e], da, ea);
                            eb = fma(U[e], db, eb);
                        }
                    }
                    if (A.grad) {
                        ea = adj_wave_sum(ea);
                        eb = adj_wave_sum(eb);
                        if ((tid & 63) == 0) {
                            atomicAdd(&s_ge[0][(ib + i) / X.kb], ea);
                            atomicAdd(&s_ge[1][(ib + i) % X.kb], eb);
                        }
                    }
                }
            }
        }
        if (A.grad) {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const double va = adj_wave_sum(cA[ax]), vb = adj_wave_sum(cB[ax]);
                if ((tid & 63) == 0) {
                    atomicAdd(&s_gc[0][ax], va);
                    atomicAdd(&s_gc[1][ax], vb);
                }
            }
        }
    }
    // the share of L in a fixed order
    s_red[tid] = energy;
    __syncthreads();
    for (int w = NT / 2; w > 0; w >>= 1) {
        if (tid < w) s_red[tid] += s_red[tid + w];
        __syncthreads();
    }
    if (tid == 0 && W.share >= 0) {
        A.energy[2 * (int64_t)W.share] = s_red[0];
        A.energy[2 * (int64_t)W.share + 1] = 0.0;
    }
    if (!A.grad) return;
    double* g = A.part + (int64_t)(blockIdx.x % (unsigned)A.n_slices) * A.slice_stride;
    const eri_shell_pair X = P[W.side];
    if (tid < 6) unsafeAtomicAdd(g + 3 * (int64_t)(tid < 3 ? X.sa : X.sb) + tid % 3, s_gc[tid / 3][tid % 3]);
    if (tid < 2 * ERI_MAX_K) {
        const int q = tid / ERI_MAX_K, k = tid % ERI_MAX_K;
        if (k < (q ? X.kb : X.nprim / X.kb)) unsafeAtomicAdd(g + A.ns3 + A.poff[q ? X.sb : X.sa] + k, s_ge[q][k]);
    }
}

}  // namespace

// Launches of a list: 64 threads a workgroup where the larger side's U has at
// most ADJ_NARROW values, else 256; each launch has as much LDS as its largest
// class needs.
constexpr int ADJ_NARROW = 512;

struct eri_adj_state {
    eri_item* d_items = nullptr;
    adj_class* d_cls = nullptr;
    adj_work* d_work = nullptr;
    int64_t n_shares = 0;
    // the launches: 256 threads and 64, each the work with a share of L first (an L alone needs no other)
    int64_t first[2] = {0, 0};
    int n0[2] = {0, 0}, n[2] = {0, 0};
    int lds[2] = {0, 0};               // bytes
    int64_t* d_bf = nullptr;
    int64_t* d_poff = nullptr;
    double* d_energy = nullptr;
    double* d_part = nullptr;
    int64_t nbf = 0, n_grad = 0;
    int n_slices = 1;
};

void eri_adj_free(eri_adj_state* s)
{
    if (!s) return;
    void* ptrs[] = {s->d_items, s->d_cls, s->d_work, s->d_bf, s->d_poff, s->d_energy, s->d_part};
    for (void* x : ptrs)
        if (x) (void)hipFree(x);
    delete s;
}

// Which classes of a list come here, and for which of them L does too, from
// what they cost here and through the derived classes (us).
//   A gradient costs a class here its primitive quartets, at a rate that is the
// same from some ten thousand of them on.  Through the derived classes it is
// some 30 launches and waits, a chain of launches that each last as long as the
// deepest contraction, and a smaller rate, which a d-d pair (g-d pairs among its
// derived ones) raises by a share per derived item.  Measured here / there in ms:
// 2048 quartets of K = 1 [pp|pp] 0.13 / 0.51, [dd|dd] 0.34 / 1.5; of K 1..3 0.49 / 0.88
// and 2.9 / 3.8; 1024 of K = 6 [ps|ps] 3.3 / 5.2, [pp|pp] 14.0 / 6.1, [dp|dp] 35.8 / 12.8;
// 256 of K = 6 0.85 / 5.1, 3.7 / 5.5, 9.7 / 8.7; 256 of K = 10 [ss|ss] 3.5 / 28, [pp|pp]
// 26 / 36, [dp|dp] 69 / 61.  Over the 36 classes of pair types, 64 to 2048 quartets
// and K up to 10 the choice costs at most 16% of the better time.
//   L alone is some half of the work here (one launch for all classes, so that
// only the longest chain over the source pairs counts), and there one launch of
// each class's own kernel: 2048 quartets of K = 1 [pp|pp] 55 / 23 us, [dd|dd] 160 / 45;
// of K 1..3 [ss|ss] 74 / 59, [pp|pp] 245 / 57, [dd|dd] 1474 / 159; 4 of them 33 / 55, 85 / 50,
// 303 / 110; 256 of K = 6 281 / 704, 1812 / 570, 13800 / 1650.  Calls with and without a
// gradient take L from the same place, so that it has the same bits in both;
// with a gradient it is a by-product here and costs a second stream there (12 us,
// or up to a seventh of a launch that fills the chip).  So it comes from there
// only where that is clearly the cheaper place for all of the list: of 191 lists
// of one class L alone then takes 0.56 of the time that it takes here, and at most
// twice that of the class's own kernel.
//   Above ERI_ADJ_MAX quartets stand the rates that the line was drawn by: 4096 /
// 16384 of K 1..3 [pp|pp] 0.89 / 3.28 and 0.94 / 1.50 ms, [dp|dp] 2.41 / 9.21 and 1.83 / 4.13.
constexpr int64_t ERI_ADJ_MAX = 2048;

void eri_adj_routes(eri_plan* p)
{
    // ns per primitive quartet by the types of the two pairs: ss, ps, pp, ds, dp, dd
    static const double rates[6][6] = {{1.4, 1.7, 3.3, 3.1, 8.8, 13.5},     {1.7, 2.4, 4.8, 4.6, 9.7, 14.5},
                                       {3.3, 4.8, 10.3, 10.0, 12.9, 27.7},  {3.1, 4.6, 10.0, 9.7, 12.8, 27.5},
                                       {8.8, 9.7, 12.9, 12.8, 26.9, 37.6},  {13.5, 14.5, 27.7, 27.5, 37.6, 77.0}};
    // us per primitive quartet of a chain through a class's own kernel, by the smaller pair
    static const double step[6] = {0.22, 0.31, 0.45, 0.45, 0.78, 1.24};
    auto type = [](int x, int y) {
        const int hi = std::max(x, y), lo = std::min(x, y);
        return hi == 0 ? 0 : hi == 1 ? 1 + lo : 3 + lo;
    };
    double work = 0.0, longest = 0.0, energy_there = 0.0;
    for (int c = 0; c < 256; ++c) {
        p->adj_listed[c] = p->adj_energy[c] = false;
        const int L[4] = {c >> 6, (c >> 4) & 3, (c >> 2) & 3, c & 3};
        if (p->class_count[c] == 0 || p->class_count[c] > ERI_ADJ_MAX || *std::max_element(L, L + 4) > 2) continue;
        const int x = type(L[0], L[1]), y = type(L[2], L[3]);
        const double rate = rates[x][y], n = (double)p->class_count[c], pq = p->class_pq[c], deep = (double)p->class_maxpq[c];
        const double ne = (double)(adj_nc(L[0]) * adj_nc(L[1]) * adj_nc(L[2]) * adj_nc(L[3]));
        const double items = 6.0 + 8.0 * std::sqrt(std::sqrt(pq / n));   // derived items of a quartet
        p->adj_listed[c] = 1e-3 * rate * pq < 430.0 + 0.4 * ne + (2.6 + 0.005 * ne) * deep + 1.8e-5 * ne * pq +
                                                  (std::max(x, y) == 5 ? 0.015 * items * n : 0.0);
        if (!p->adj_listed[c]) continue;
        work += 1e-3 * (0.1 + 0.54 * rate) * pq + 5e-3 * n;
        longest = std::max(longest, (1.7 + 0.48 * rate) * std::sqrt(deep));
        // (up to L_tot = 2 a lane walks the contraction, else a slot of lanes)
        energy_there += 32.0 + (L[0] + L[1] + L[2] + L[3] <= 2 ? 0.58 : step[std::min(x, y)]) * deep + 1e-5 * ne * n +
                        5e-7 * ne * pq;
    }
    const bool here = 10.0 + std::max(work, longest) <= energy_there;
    for (int c = 0; c < 256; ++c) p->adj_energy[c] = here && p->adj_listed[c];
}

static int adj_build(eri_plan* p, eri_adj_state* st)
{
    const int64_t nq = p->n_quartets, ns = (int64_t)p->sh_L.size();
    auto listed = [&](int64_t q) {
        const int32_t* u = p->quartets.data() + 4 * q;
        return p->adj_listed[p->sh_L[u[0]] * 64 + p->sh_L[u[1]] * 16 + p->sh_L[u[2]] * 4 + p->sh_L[u[3]]];
    };
    // the record of an ordered shell pair: the plan holds one of its two orders
    std::vector<eri_item> items(nq);
    const std::vector<uint64_t>& keys = p->pair_keys;
    auto record = [&](int32_t x, int32_t y, int32_t& out) {
        for (int rev = 0; rev < 2; ++rev) {
            const uint64_t k = rev ? ((uint64_t)(uint32_t)y << 32) | (uint32_t)x : ((uint64_t)(uint32_t)x << 32) | (uint32_t)y;
            const auto it = std::lower_bound(keys.begin(), keys.end(), k);
            if (it != keys.end() && *it == k) {
                out = (int32_t)((uint32_t)(it - keys.begin()) | (rev ? 0x80000000u : 0u));
                return true;
            }
        }
        return false;
    };
    for (int64_t q = 0; q < nq; ++q) {
        const int32_t* u = p->quartets.data() + 4 * q;
        items[q].bra = items[q].ket = 0;
        if (!listed(q)) continue;
        if (!record(u[0], u[1], items[q].bra) || !record(u[2], u[3], items[q].ket)) return ERI_ESTATE;
    }
    std::vector<adj_class> cls;
    struct entry {
        adj_work w;
        double cost;
    };
    std::vector<entry> work[2];
    int64_t targets = 0;
    for (int64_t q = 0; q < nq; ++q)
        if (listed(q)) {
            const int32_t* u = p->quartets.data() + 4 * q;
            targets += (int64_t)p->sh_K[u[0]] * p->sh_K[u[1]] + (int64_t)p->sh_K[u[2]] * p->sh_K[u[3]];
        }
    const int per = (int)std::min<int64_t>(256, std::max<int64_t>(1, targets / ADJ_WORK));
    for (int c = 0; c < 256; ++c) {
        if (!p->adj_listed[c]) continue;
        adj_class e;
        std::memset(&e, 0, sizeof(e));
        const int L[4] = {c >> 6, (c >> 4) & 3, (c >> 2) & 3, c & 3};
        std::copy(L, L + 4, e.L);
        e.first = p->class_qoff[c];
        e.eoff = p->class_eoff[c];
        const int lb = L[0] + L[1], lk = L[2] + L[3];
        const int u[2] = {adj_nc(L[0]) * adj_nc(L[1]) * adj_nherm(lb + 2), adj_nc(L[2]) * adj_nc(L[3]) * adj_nherm(lk + 2)};
        // up to four source pairs a batch, within 60 KB (two workgroups a CU; (dd|dd) takes one pair)
        e.jc = 4;
        while (e.jc > 1 && adj_lds(L, e.jc).end * 8 > 60 * 1024) e.jc /= 2;
        const int k = std::max(u[0], u[1]) <= ADJ_NARROW ? 1 : 0;
        const bool shares = p->adj_energy[c];
        st->lds[k] = std::max(st->lds[k], adj_lds(L, e.jc).end * 8);
        for (int64_t q = e.first; q < e.first + p->class_count[c]; ++q) {
            int np[2];
            for (int side = 0; side < 2; ++side) {
                const uint64_t key = keys[(side ? items[q].ket : items[q].bra) & 0x7fffffff];
                np[side] = p->sh_K[key >> 32] * p->sh_K[key & 0xffffffffu];
            }
            for (int side = 0; side < 2; ++side)
                for (int i = 0; i < np[side]; i += per) {
                    entry x;
                    x.w = adj_work{(int32_t)q, (int32_t)cls.size(), (int16_t)side, (int16_t)i,
                                   (int16_t)std::min(per, np[side] - i), 0, side == 0 && shares ? 0 : -1};
                    const double step = (double)u[side] * adj_nherm(side ? lb : lk) / (k ? 64 : 256) + 1000.0;
                    x.cost = x.w.in * (double)np[side ^ 1] * step;
                    work[k].push_back(x);
                }
        }
        cls.push_back(e);
    }
    std::vector<adj_work> list;
    for (int k = 0; k < 2; ++k) {
        // those with a share of L first, then the longest first
        std::stable_sort(work[k].begin(), work[k].end(), [](const entry& x, const entry& y) {
            return x.w.share != y.w.share ? x.w.share > y.w.share : x.cost > y.cost;
        });
        st->first[k] = (int64_t)list.size();
        st->n[k] = (int)work[k].size();
        for (entry& x : work[k])
            if (x.w.share >= 0) {
                x.w.share = (int32_t)st->n_shares++;
                ++st->n0[k];
            }
        for (const entry& x : work[k]) list.push_back(x.w);
    }
    std::vector<int64_t> bf(ns + 1, 0);
    for (int64_t s = 0; s < ns; ++s) bf[s + 1] = bf[s] + ncart(p->sh_L[s]);
    st->nbf = bf[ns];
    st->n_grad = 3 * ns + (int64_t)p->sh_exps.size();
    st->n_slices = (int)std::max<int64_t>(1, std::min<int64_t>(ADJ_SLICES_MAX, ADJ_SLICE_DOUBLES / std::max<int64_t>(1, st->n_grad)));
    ERI_TRY(upload(p, (void**)&st->d_items, items.empty() ? nullptr : items.data(), items.size() * sizeof(eri_item)));
    ERI_TRY(upload(p, (void**)&st->d_cls, cls.empty() ? nullptr : cls.data(), cls.size() * sizeof(adj_class)));
    ERI_TRY(upload(p, (void**)&st->d_work, list.empty() ? nullptr : list.data(), list.size() * sizeof(adj_work)));
    ERI_TRY(upload(p, (void**)&st->d_bf, bf.data(), bf.size() * sizeof(int64_t)));
    ERI_TRY(upload(p, (void**)&st->d_poff, p->sh_off.empty() ? nullptr : p->sh_off.data(), p->sh_off.size() * sizeof(int64_t)));
    ERI_TRY(upload(p, (void**)&st->d_energy, nullptr, 2 * (size_t)st->n_shares * sizeof(double)));
    ERI_TRY(upload(p, (void**)&st->d_part, nullptr, (size_t)st->n_slices * st->n_grad * sizeof(double)));
    return ERI_OK;
}

int eri_adj_backward(eri_plan* p, hipStream_t strm, const double* dl, const double* density, int64_t nbf, double* grad_c,
                     double* grad_e, double* energy)
{
    if (!p->adj) {
        eri_adj_state* st = new (std::nothrow) eri_adj_state();
        if (!st) return ERI_ENOMEM;
        int rc;
        try {
            rc = adj_build(p, st);
        } catch (const std::bad_alloc&) {
            rc = ERI_ENOMEM;
        }
        if (rc != ERI_OK) {
            eri_adj_free(st);
            return rc;
        }
        p->adj = st;
    }
    eri_adj_state* st = p->adj;
    if (density && nbf != st->nbf) return ERI_EINVAL;
    adj_args a;
    std::memset(&a, 0, sizeof(a));
    a.items = st->d_items;
    a.pairs = p->d_pairs;
    a.prims = p->d_prims;
    a.grad = grad_c != nullptr;
    a.dl = dl;
    a.dens = density;
    a.bf = st->d_bf;
    a.nbf = nbf;
    a.poff = st->d_poff;
    a.part = st->d_part;
    a.slice_stride = st->n_grad;
    a.ns3 = 3 * (int64_t)p->sh_L.size();
    a.n_slices = st->n_slices;
    a.energy = st->d_energy;
    if (grad_c) ERI_TRY(eri_grad_zero(st->d_part, st->n_slices * st->n_grad, strm));
    a.cls = st->d_cls;
    for (int k = 0; k < 2; ++k) {
        const int n = grad_c ? st->n[k] : st->n0[k];
        if (!n) continue;
        a.work = st->d_work + st->first[k];
        void* args[] = {&a};
        const void* fn = k ? (const void*)adj_list_kernel<64> : (const void*)adj_list_kernel<256>;
        ERI_HIP_TRY(hipLaunchKernel(fn, dim3(n), dim3(k ? 64 : 256), args, st->lds[k], strm));
    }
    if (grad_c) ERI_TRY(eri_grad_reduce(st->d_part, st->n_slices, st->n_grad, a.ns3, grad_c, grad_e, strm));
    if (energy && st->n_shares) ERI_TRY(eri_energy_add(st->d_energy, st->n_shares, energy, strm));
    return ERI_OK;
}
