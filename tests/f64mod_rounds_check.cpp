// The rounds of the double-precision transforms on the host, with the reductions where the kernels have them, next to the same
// rounds in exact integers.  Twiddles are centred representatives.
#include <stddef.h>
#include <stdint.h>

#include "../paper_2604_16834_amd/csrc/f64mod.h"

typedef __int128 i128;

static double mul(double y, int64_t w, double q, double qinv, int value_only) {
    return value_only ? f64m_mulmod_any(y, (double)w, q, qinv) : f64m_mulmod(y, (double)w, (double)w / q, q);
}
static uint64_t residue(i128 v, uint64_t q) {
    i128 m = v % (i128)q;
    return (uint64_t)(m < 0 ? m + q : m);
}

extern "C" {

// `stages` stages on eight values (two groups of four for two stages, as at the end of the forward and the start of the inverse
// transform): fwd with f64m_fwd_begin where `begin`; inv with f64m_inv_mid (three stages) and f64m_inv_end where `end` (two
// stages: the sums of sums reduced where `end`).  io: the values as doubles; tw: 7 twiddles ((1 << a) - 1 + group), the second
// group of four takes its own three at tw + 3.  worst[0] = largest multiplicand, worst[1] = largest magnitude of any sum, in
// units of q; want: the results modulo q.  Returns the number of results that are not congruent or not integers.
long run_round(double* io, const int64_t* tw, uint64_t q, int stages, int inverse, int begin, int end, int value_only, double* worst,
               size_t n) {
    const double qd = (double)q, qinv = 1.0 / qd;
    long bad = 0;
    worst[0] = worst[1] = 0.0;
    for (size_t i = 0; i < n; i++) {
        double* v = io + 8 * i;
        const int64_t* t7 = tw + 7 * i;
        uint64_t want[8];
        const int span = 1 << stages;
        {
            i128 r[8];
            for (int j = 0; j < 8; j++) r[j] = residue((i128)v[j], q);
            for (int g = 0; g < 8; g += span)
                for (int s = 0; s < stages; s++) {
                    const int a = inverse ? stages - 1 - s : s, half = span >> (a + 1);
                    for (int rr = 0; rr < span; rr++) {
                        if (rr & half) continue;
                        const i128 w = t7[(g ? 3 : 0) + (1 << a) - 1 + (rr >> (stages - a))];
                        i128 &x = r[g + rr], &y = r[g + rr + half];
                        const i128 t = inverse ? (x - y) * w % (i128)q : y * w % (i128)q;
                        const i128 s0 = inverse ? x + y : x + t, s1 = inverse ? t : x - t;
                        x = residue(s0, q);
                        y = residue(s1, q);
                    }
                }
            for (int j = 0; j < 8; j++) want[j] = (uint64_t)r[j];
        }
        if (begin) f64m_fwd_begin(v, qd, qinv);
        for (int s = 0; s < stages; s++) {
            const int a = inverse ? stages - 1 - s : s, half = span >> (a + 1);
            for (int g = 0; g < 8; g += span)
                for (int rr = 0; rr < span; rr++) {
                    if (rr & half) continue;
                    const int64_t w = t7[(g ? 3 : 0) + (1 << a) - 1 + (rr >> (stages - a))];
                    double &x = v[g + rr], &y = v[g + rr + half];
                    const double m = inverse ? x - y : y;
                    if (__builtin_fabs(m) / qd > worst[0]) worst[0] = __builtin_fabs(m) / qd;
                    const double t = mul(m, w, qd, qinv, value_only);
                    const double s0 = inverse ? x + y : x + t, s1 = inverse ? t : x - t;
                    x = s0;
                    y = s1;
                    if (__builtin_fabs(x) / qd > worst[1]) worst[1] = __builtin_fabs(x) / qd;
                    if (__builtin_fabs(y) / qd > worst[1]) worst[1] = __builtin_fabs(y) / qd;
                }
            if (inverse && stages == 3 && s == 0) f64m_inv_mid<1>(v, qd, qinv);
        }
        if (inverse && end && stages == 3) f64m_inv_end(v, qd, qinv);
        if (inverse && end && stages == 2) {
            v[0] = f64m_reduce(v[0], qd, qinv);
            v[4] = f64m_reduce(v[4], qd, qinv);
        }
        for (int j = 0; j < 8; j++)
            if ((double)(int64_t)v[j] != v[j] || residue((i128)(int64_t)v[j], q) != want[j]) bad++;
    }
    return bad;
}

// The sum of a fused inner product over `digits` digits but `own` (none left out where own >= digits), then two products that
// need not be of reduced values (the own limb's, a product's addend): io holds n rows of digits + 2 multiplicands, each
// negated where its product is negative, so that the sum grows as far as it can; w the multipliers in [0, q).  worst: the largest
// magnitude of a sum in units of q.  Returns the number of sums that are wrong.
long run_key_sum(double* io, const uint64_t* w, uint64_t q, int digits, int own, double* worst, size_t n) {
    const double qd = (double)q, qinv = 1.0 / qd;
    long bad = 0;
    *worst = 0.0;
    for (size_t i = 0; i < n; i++) {
        double* y = io + (digits + 2) * i;
        const uint64_t* k = w + (digits + 2) * i;
        double acc = 0.0;
        i128 want = 0;
        auto add = [&](int j) {
            double t = f64m_mulmod_any(y[j], (double)k[j], qd, qinv);
            if (t < 0.0) y[j] = -y[j], t = f64m_mulmod_any(y[j], (double)k[j], qd, qinv);
            acc += t;
            want = (want + (i128)y[j] * (i128)k[j]) % (i128)q;
            if (acc / qd > *worst) *worst = acc / qd;
        };
        int j = own == 0 ? 1 : 0;
        while (j < digits) {
            int jn = j + 1;
            if (jn == own) jn++;
            add(j);
            if (f64m_sum_due((uint32_t)j, (uint32_t)jn)) {
                acc = f64m_reduce(acc, qd, qinv);
                if (acc < 0.0) {  // the negated sum: as good a sum of negated terms, and the one that grows
                    acc = -acc;
                    want = -want;
                }
            }
            j = jn;
        }
        add(digits);
        add(digits + 1);
        if (f64m_canonical(f64m_reduce(acc, qd, qinv), qd) != residue(want, q)) bad++;
    }
    return bad;
}

}  // extern "C"
