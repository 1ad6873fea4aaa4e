// Device structures and helpers of the adjoint's density form (Hermite
// Coulomb kernels, generated by codegen_coulomb.py).
#pragma once
#include "eri_device.h"

// L's bits must not depend on which products the compiler fuses: every fma of
// these kernels is written out.
#pragma clang fp contract(off)

// Source primitive pairs [lo, hi) of the targets of one shell pair (indices
// into the plan's primitive-pair table).
struct eri_coul_range {
    int32_t lo, hi;
};

// One wavefront's work: n <= 64 consecutive target primitive pairs against
// the source primitive pairs [lo, hi) of one class; each target takes part
// with those of its shell pair's range.
struct eri_coul_job {
    int64_t trec, srec;      // records of target t0 and of source s0 (doubles into rec)
    int64_t tpot;            // V_0 of target t0 (doubles into pot)
    int64_t range;           // ranges[range + shell pair]
    int32_t t0, n;           // first target primitive pair, targets
    int32_t lo, hi, s0;      // sources (global indices) and the class's first
    int32_t pot_stride;      // doubles from V_k to V_(k+1) of a target
};

struct eri_coul_args {
    const eri_coul_job* jobs;
    int64_t n_jobs;
    const double* full;              // per primitive pair: p, P, (-1)^|t| H_t
    const double* rec;               // the same, -p and zeros where an H_t is not finite
    const eri_coul_range* ranges;
    const int32_t* prim_pair;        // shell pair of each primitive pair
    double* pot;
    double* energy;                  // per job: its share of L, (high, low)
};

const void* eri_coul_kernel(int lt, int ls, int grad);

// Error-free sum of two doubles (Knuth's two-sum): s + e == a + b exactly.
ERI_DEV void eri_two_sum(double a, double b, double& s, double& e)
{
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

ERI_DEV void eri_coul_add(double& hi, double& lo, double x)
{
    double e;
    eri_two_sum(hi, x, hi, e);
    lo += e;
}

// 1/sqrt(x) of an ordinary positive double: the hardware estimate and two
// Newton steps.
ERI_DEV double eri_coul_rsqrt(double x)
{
    double r = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int k = 0; k < 2; ++k) r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
    return r;
}

// The nine table columns that F_MMAX's Taylor series reads, into LDS (26 KB):
// the rows that the lanes of a wavefront read lie apart, and a gather of 64
// lines a load from the cache costs more than the recurrences it feeds.
template <int MMAX>
ERI_DEV void eri_coul_stage_boys(double* __restrict__ s)
{
    for (int i = threadIdx.x; i < 361 * 9; i += blockDim.x) {
        const int k = i / 9, c = i - 9 * k;
        s[i] = eri_boys_table[k * ERI_BOYS_NCOL + MMAX + c];
    }
    __syncthreads();
}

// eri_boys with the staged columns.
template <int MMAX>
ERI_DEV void eri_boys_lds(double T, double* __restrict__ F, const double* __restrict__ s)
{
    const double et = exp(-T);
    if (T < ERI_BOYS_TMAX) {
        const int k = __double2int_rn(T * (1.0 / ERI_BOYS_DT));
        const double d = fma((double)k, ERI_BOYS_DT, -T);
        const double* __restrict__ row = s + 9 * k;
        double v = row[8];
        v = fma(v, d * (1.0 / 8.0), row[7]);
        v = fma(v, d * (1.0 / 7.0), row[6]);
        v = fma(v, d * (1.0 / 6.0), row[5]);
        v = fma(v, d * (1.0 / 5.0), row[4]);
        v = fma(v, d * (1.0 / 4.0), row[3]);
        v = fma(v, d * (1.0 / 3.0), row[2]);
        v = fma(v, d * (1.0 / 2.0), row[1]);
        v = fma(v, d, row[0]);
        F[MMAX] = v;
#pragma unroll
        for (int m = MMAX - 1; m >= 0; --m) F[m] = fma(2.0 * T, F[m + 1], et) * (1.0 / (double)(2 * m + 1));
    } else {
        const double ir = eri_coul_rsqrt(T);
        F[0] = 0.88622692545275801365 * ir;   // sqrt(pi)/2 / sqrt(T)
        const double h = 0.5 * ir * ir;
#pragma unroll
        for (int m = 0; m < MMAX; ++m) F[m + 1] = fma((double)(2 * m + 1), F[m], -et) * h;
    }
}

// The wavefront's shares of L, added in a fixed order; lane 0 writes them.
ERI_DEV void eri_coul_job_sum(double hi, double lo, double* __restrict__ out)
{
    for (int o = 32; o > 0; o >>= 1) {
        const double h2 = __shfl_xor(hi, o), l2 = __shfl_xor(lo, o);
        // both lanes of a pair must form the same sum
        const bool low = (threadIdx.x & o) == 0;
        double e;
        eri_two_sum(low ? hi : h2, low ? h2 : hi, hi, e);
        lo = (low ? lo : l2) + (low ? l2 : lo) + e;
    }
    if ((threadIdx.x & 63) == 0) {
        out[0] = hi;
        out[1] = lo;
    }
}
