"""Generator of the Hermite Coulomb kernels of the adjoint's density form.

With Gbar = D_ab D_cd the scalar L = sum w D_ab D_cd (ab|cd) is a quadratic
form in the charge of every primitive pair,
    rho_i(r) = sum_ab D_ab (primitive pair i of ab) = sum_t H_i[t] Lambda_t(r),
expanded in Hermite Gaussians Lambda_t = d^t/dP^t exp(-p |r - P|^2), |t| <= La
+ Lb (McMurchie and Davidson's scheme).  What is needed of all quartets that a
pair takes part in is then its potential in the same basis,
    V_i[t] = sum_j 2 pi^(5/2) / sqrt(p + q) sum_t' (-1)^|t'| H_j[t'] R_(t+t')(P - Q),
with R the Hermite Coulomb integrals of exponent rho = p q / (p + q): L is the
sum of H_i V_i, and since the derivatives of a pair's Gaussians with respect
to its centres and exponents are Gaussian products with up to two more units
of angular momentum, its gradient needs V_i[t] up to |t| = La + Lb + 2 and
nothing else.  No integral over four shells and no derived shell appears.

One kernel per (LT, LS) = (La + Lb of the target pair, Lc + Ld of the source
pair), with (grad) or without the two additional orders of V.
"""

LMAX = 4   # La + Lb of a pair of shells up to d


def hermites(L):
    """(t, u, v) with t + u + v <= L, by order, x first within one."""
    return [(t, u, s - t - u) for s in range(L + 1) for t in range(s, -1, -1) for u in range(s - t, -1, -1)]


def kernel_name(lt, ls, grad):
    return "eri_coul_%d%d%s" % (lt, ls, "g" if grad else "e")


def emit_kernel(lt, ls, grad):
    """Each lane holds one target primitive pair; the wavefront walks the
    source pairs of its job, whose record (exponent, centre, signed Hermite
    coefficients) is the same for every lane: scalar loads and scalar operands.
    A lane meets the sources outside its target's range with a factor of zero,
    but for those with an infinite or NaN charge, which it would carry into the
    potential of a target that shares no quartet with them: the first loop reads
    records where their charges are zero and their exponent is negative, and a
    second loop, entered where there are such, takes them from the full records
    and skips them lane by lane.  (Skipping all sources so splits the loop's body:
    4 atoms, whose wavefronts are alone on their SIMD, 1315 us, 1924 so; a branch
    around the marked ones 1358.)
    R is built along z for each (x, y), along y for each x, then x, so that
    besides V only three pairs of columns are live, and every R_k at m = 0 is
    used for all t + t' = k at once.  The potentials of orders up to LT are
    summed per source first: their product with the target's coefficients is
    the interaction's share of L, added with two-sum compensation.
    Both forms evaluate the Boys function to the same order and use the same
    fma chains for L, so that L has the same bits with and without a gradient."""
    N = lt + ls + 2
    top = lt + 2 if grad else lt
    T, S = hermites(lt), hermites(ls)
    V = hermites(top)
    tix = {t: k for k, t in enumerate(V)}
    low = set(T)
    name = kernel_name(lt, ls, grad)
    o = []
    em = o.append

    def loop(skip):
        em("    for (int j = job.lo; j < job.hi; ++j) {")
        em("        const int64_t sj = job.srec + (int64_t)(j - job.s0) * %d;" % (4 + len(S)))
        if skip:
            em("        const double* __restrict__ sr = A.full + sj;")
            em("        if (__double_as_longlong(A.rec[sj]) >= 0 || j < lo || j >= hi) continue;")
            em("        const double q = sr[0];")
        else:
            em("        const double* __restrict__ sr = A.rec + sj;")
            em("        left |= __double_as_longlong(sr[0]);")
            em("        const bool in = j >= lo && j < hi;")
            em("        const double q = fabs(sr[0]);")
        em("        const double X = Px - sr[1], Y = Py - sr[2], Z = Pz - sr[3];")
        em("        const double ir = eri_coul_rsqrt(p + q);")
        em("        const double rho = p * q * ir * ir;")
        em("        const double pref = %sERI_TWO_PI_52 * ir%s;" % (("", "") if skip else ("in ? ", " : 0.0")))
        em("        double F[%d];" % (N + 1))
        em("        eri_boys_lds<%d>(rho * fma(X, X, fma(Y, Y, Z * Z)), F, s_boys);" % N)
        em("        const double b = -2.0 * rho;")
        em("        double f = pref;")
        # the order of V plus the source's order is what R is needed to
        M = top + ls
        for m in range(M + 1):
            em("        const double x0_%d = f * F[%d];%s" % (m, m, " f *= b;" if m < M else ""))
        for k in range(len(T)):
            em("        double c%d = 0.0;" % tix[T[k]])
        sidx = {s: k for k, s in enumerate(S)}

        def scatter(k, val):
            for t in V:
                s = (k[0] - t[0], k[1] - t[1], k[2] - t[2])
                if min(s) < 0 or sum(s) > ls:
                    continue
                dst = ("c%d" if t in low else "V%d") % tix[t]
                em("        %s = fma(sr[%d], %s, %s);" % (dst, 4 + sidx[s], val, dst))

        def step(dst, ax, n, a, b2, m):
            # R^m_(n+1) = n R^(m+1)_(n-1) + X R^(m+1)_n along one axis
            if n == 0:
                em("        const double %s_%d = %s * %s_%d;" % (dst, m, ax, a, m + 1))
            elif n == 1:
                em("        const double %s_%d = fma(%s, %s_%d, %s_%d);" % (dst, m, ax, a, m + 1, b2, m + 1))
            else:
                em("        const double %s_%d = fma(%s, %s_%d, %.1f * %s_%d);" % (dst, m, ax, a, m + 1, float(n), b2, m + 1))

        for t in range(M + 1):
            if t > 0:
                for m in range(M - t + 1):
                    step("x%d" % t, "X", t - 1, "x%d" % (t - 1), "x%d" % (t - 2), m)
            for u in range(M - t + 1):
                yu = "y%d_%d" % (t, u)
                if u == 0:
                    for m in range(M - t + 1):
                        em("        const double %s_%d = x%d_%d;" % (yu, m, t, m))
                else:
                    for m in range(M - t - u + 1):
                        step(yu, "Y", u - 1, "y%d_%d" % (t, u - 1), "y%d_%d" % (t, u - 2), m)
                for v in range(M - t - u + 1):
                    zv = "z%d_%d_%d" % (t, u, v)
                    if v == 0:
                        for m in range(M - t - u + 1):
                            em("        const double %s_%d = %s_%d;" % (zv, m, yu, m))
                    else:
                        for m in range(M - t - u - v + 1):
                            step(zv, "Z", v - 1, "z%d_%d_%d" % (t, u, v - 1), "z%d_%d_%d" % (t, u, v - 2), m)
                    scatter((t, u, v), zv + "_0")
        em("        double e = h0 * c0;")
        for k in range(1, len(T)):
            em("        e = fma(h%d, c%d, e);" % (k, k))
        em("        eri_coul_add(e_hi, e_lo, %s);" % ("e" if skip else "in ? e : 0.0"))
        if grad:
            for k in range(len(T)):
                em("        V%d += c%d;" % (k, k))
        em("    }")

    em("// target pairs of order %d, source pairs of order %d" % (lt, ls))
    em("__global__ __launch_bounds__(256) void %s(eri_coul_args A)" % name)
    em("{")
    em("    __shared__ double s_boys[%d];" % (361 * 9))
    em("    eri_coul_stage_boys<%d>(s_boys);" % N)
    em("    const int64_t jb = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));")
    em("    if (jb >= A.n_jobs) return;")
    em("    const eri_coul_job job = A.jobs[jb];")
    em("    const int lane = threadIdx.x & 63;")
    em("    const bool active = lane < job.n;")
    em("    const int it = active ? lane : 0;")
    em("    const double* __restrict__ tr = A.full + job.trec + (int64_t)it * %d;" % (4 + len(T)))
    em("    const double p = tr[0], Px = tr[1], Py = tr[2], Pz = tr[3];")
    for k in range(len(T)):
        sign = "-" if sum(T[k]) % 2 else ""      # the record carries (-1)^|t| H[t]
        em("    const double h%d = %str[%d];" % (k, sign, 4 + k))
    em("    const eri_coul_range rg = A.ranges[job.range + A.prim_pair[job.t0 + it]];")
    em("    const int lo = rg.lo, hi = active ? rg.hi : 0;")
    if grad:
        for k in range(len(V)):
            em("    double V%d = 0.0;" % k)
    em("    double e_hi = 0.0, e_lo = 0.0;")
    em("    long long left = 0;   // negative once a marked source has come")
    loop(False)
    em("    if (left < 0) {")
    loop(True)
    em("    }")
    if grad:
        em("    if (active) {")
        em("        double* out = A.pot + job.tpot + lane;")
        em("        const int64_t st = job.pot_stride;")
        for k in range(len(V)):
            em("        unsafeAtomicAdd(out + %d * st, V%d);" % (k, k))
        em("    }")
    em("    eri_coul_job_sum(e_hi, e_lo, A.energy + 2 * jb);")
    em("}")
    return "\n".join(o) + "\n"


def generate():
    """Source of the kernels' translation unit."""
    parts = ["// Generated by codegen_coulomb.py -- Hermite Coulomb kernels of the adjoint's density form.",
             '#include "eri_coulomb.h"', ""]
    for lt in range(LMAX + 1):
        for ls in range(LMAX + 1):
            for grad in (True, False):
                parts.append(emit_kernel(lt, ls, grad))
    parts.append("const void* eri_coul_kernel(int lt, int ls, int grad)\n{")
    parts.append("    static const void* const k[2][%d][%d] = {" % (LMAX + 1, LMAX + 1))
    for grad in (False, True):
        parts.append("        {%s}," % ", ".join(
            "{%s}" % ", ".join("(const void*)%s" % kernel_name(lt, ls, grad) for ls in range(LMAX + 1))
            for lt in range(LMAX + 1)))
    parts.append("    };\n    return k[grad ? 1 : 0][lt][ls];\n}\n")
    return "\n".join(parts)
