// Which kernel takes a basis conversion between two transforms, by its sizes alone.  No dependency but <stdint.h>: a CPU test goes through every
// size that a context can have.  The launchers instantiate exactly the kernels named here and refuse every other size.
#pragma once
#include <stdint.h>

#define CONV_MID_TERMS 9  // most source limbs that the LDS form takes through the inverse transform's second pass

// The converting first pass of a ring of 2^(11 + log_hi) points, nd source limbs in rows of ap constants: the terms that it is instantiated
// with (nd or more; what is beyond nd multiplies the row's zeros), 0: there is no such kernel.
constexpr uint32_t hi_conv_terms(uint32_t log_hi, uint32_t ap, uint32_t nd) {
    if (log_hi < 2 || log_hi > 6 || nd == 0 || nd > ap || (ap != 4 && ap != 8 && ap != 12 && ap != 16)) return 0;
    if (log_hi < 4) {  // what the columns do not take (mid_conv_per): more than ten source limbs on rings of 2^13 points, five on those of 2^14
        if (log_hi == 2) return ap == 16 || (ap == 12 && nd > 10) ? ap : 0;
        return ap == 4 ? 0 : (ap == 12 && nd == 9 ? 9 : ap);
    }
    if (ap == 4 && nd == 1) return 1;  // the rescale: one dropped limb
    // as many terms as the launch has source limbs: the rest of a row is padding (digits of 7, 7 and 4 or 5
    // limbs in rows of eight: 41.0 us a launch with eight terms everywhere, 38.0 with their own).  Whole calls with two equal
    // digits at N = 2^16 take this much longer with full rows (product / activation of eight / eight rotations low in the
    // chain): digits of 2 limbs 1.02 / - / 1.04, of 3 1.02 / 1.00 / 1.02, of 5 1.03 / 1.02 / 1.03, of 6 1.04 / 1.00 / 1.03, of 7
    // 1.03 / 1.00 / 1.01, of 9 1.06 / 1.04 / 1.06, of 10 1.02 / 1.02 / 1.06, of 11 1.02 / 1.02 / 1.03, of 12 1.03 / 1.02 / 1.04
    if (ap == 4) return nd;
    if (ap == 8) return nd <= 4 ? 4 : nd;
    if (ap == 12) return nd == 9 || nd == 10 ? nd : 12;  // nine: eight special primes and the dropped limb
    return nd <= 8 ? 8 : (nd <= 10 ? 10 : (nd <= 12 ? 12 : 16));
}
// The same for the kernel that holds a column of every source limb (ntt_mid_conv_kernel)
constexpr uint32_t mid_conv_terms(uint32_t log_hi, uint32_t nd) {
    if (log_hi < 1 || log_hi > 3 || nd == 0) return 0;
    if (nd <= 5) return nd;
    if (log_hi == 3) return 0;
    if (nd <= 10) return nd;
    if (log_hi == 2) return 0;
    return nd <= 12 ? 12 : (nd <= 16 ? 16 : 0);
}
// Whether the converting kernel takes the inverse transform's second pass with it where mid_conv_per asks for that
constexpr bool conv_has_mid(uint32_t log_hi, uint32_t ap, uint32_t nd) {
    if (log_hi <= 3) return mid_conv_terms(log_hi, nd) != 0;
    const uint32_t terms = hi_conv_terms(log_hi, ap, nd);
    return terms != 0 && terms <= CONV_MID_TERMS;
}
// Whether the inverse transform's second pass goes inside the converting first pass, for a launch of `rows` (polynomial, digit) rows of nd
// source limbs (rows of ap constants) and up to n_targets targets each: 0, or the targets per workgroup.  It saves a launch with its
// round trip through memory and repeats the inverse stages per group of targets.  Measured in whole calls, one by one / together in us:
//   rescale: at every size (N = 2^13, 4 limbs 18.5 / 14.5, 2^16, 13 limbs 27.9 / 24.2; eight ciphertexts of 24 limbs the same)
//   rings up to 2^14 (ntt_mid_conv_kernel) while a thread's points of all source limbs are at most 40: one rotation at N = 2^13 of 4 + 2
//     limbs 45.6 / 33.0, of 21 + 8 50.1 / 48.9, eight 112 / 107; at 2^14 of 7 + 3 45.8 / 41.1, but of 13 + 7 (56 points) 46.1 / 49.6, of
//     21 + 8 (64) 59.9 / 66.6
//   larger rings, up to four source limbs: up to 1200 workgroups or two groups of targets (2^15, 13 + 4 limbs, one rotation 67.3 / 62.0, eight
//     276 / 275; activation of eight at 2^16 1628 / 1624, with no such line 1659); five and six: up to 300 or two groups (9 + 6 limbs
//     60.6 / 58.1, two 69.2 / 66.9, four 95.5 / 95.1, with no line 99.1); more: a single group (nothing repeated: 2^16, 3 + 8 limbs, eight
//     rotations 160 / 141), or two of four rows and more (7 + 8 limbs: one rotation 60.4 / 61.5, eight 233 / 222; with 13 + 8, four groups,
//     eight 428 / 450)
constexpr uint32_t mid_conv_per(uint32_t log_hi, uint32_t nd, uint32_t ap, uint32_t n_targets, uint32_t rows) {
    if (log_hi > 3) {
        const uint32_t groups = (n_targets + 3) / 4, wgs = groups * rows << log_hi;
        bool together = false;
        if (nd == 1) together = true;
        else if (nd <= 4) together = groups <= 2 || wgs <= 1200;
        else if (nd <= 6) together = groups <= 2 || wgs <= 300;
        else together = groups == 1 || (groups == 2 && rows >= 4);
        return together && conv_has_mid(log_hi, ap, nd) ? 4 : 0;
    }
    // rings of 2^12 points always: the passes one by one have no converting kernel there
    if (!conv_has_mid(log_hi, ap, nd) || (log_hi > 1 && nd > 1 && (nd << log_hi) > 40)) return 0;
    uint32_t per = 4;  // fewer, and more workgroups, until every CU has one
    while (per > 1 && 8 * rows * ((n_targets + per - 1) / per) < 256) per >>= 1;
    return per;
}
