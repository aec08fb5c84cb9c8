// Goes through every basis conversion that a context can ask for (all digit widths, special primes, levels and batch sizes of the rings of 2^12
// to 2^17 points) and checks that the rule names a kernel for it, wide enough and, where the rule asks for it, with the inverse pass inside; that
// sizes without a kernel are refused; and which kernels the rule can reach at all.
#include <cstdio>
#include <set>
#include <tuple>
#include "../paper_2604_16834_amd/csrc/convrule.h"

typedef uint32_t u32;
static std::set<std::tuple<u32, u32, u32, bool>> reached;  // log_hi, ap, terms, with the inverse pass (ap 0: the kernel that holds columns)
static unsigned long long n_sizes = 0;

static bool takes(u32 log_hi, u32 ap, u32 nd, u32 per) {
    n_sizes++;
    if (per && log_hi <= 3) {
        const u32 t = mid_conv_terms(log_hi, nd);
        reached.insert({log_hi, 0u, t, true});
        return t >= nd;
    }
    const u32 t = hi_conv_terms(log_hi, ap, nd);
    reached.insert({log_hi, ap, t, per != 0});
    return t >= nd && t <= ap && (!per || conv_has_mid(log_hi, ap, nd));
}
static u32 pad(u32 v) { return v <= 4 ? 4 : (v <= 8 ? 8 : 16); }

int main() {
    for (u32 log_hi = 1; log_hi <= 6; log_hi++)
        for (u32 k = 1; k <= 15; k++) {
            const u32 k_pad = pad(k), k2_pad = k + 1 > 8 && k + 1 <= 12 ? 12 : pad(k + 1);
            for (u32 level = 0; level + 1 + k <= 64; level++) {
                for (u32 n = 1; n <= 16; n++) {  // polynomials to decompose, ciphertexts to divide
                    for (u32 alpha = 1; alpha <= 16; alpha++) {
                        const u32 L1 = level + 1, E = L1 + k, nd0 = alpha < L1 ? alpha : L1, beta = (L1 + alpha - 1) / alpha;
                        const u32 per = mid_conv_per(log_hi, nd0, pad(alpha), E - nd0, n * beta), last = L1 - (beta - 1) * alpha;
                        // one launch for all digits takes the first one's kernel, a launch per digit each its own; the first digit's has to be
                        // wide enough for the last one's either way
                        const bool each = !(per && log_hi <= 3);
                        if (!takes(log_hi, pad(alpha), nd0, per) || last > nd0 || (each && !takes(log_hi, pad(alpha), last, per))) {
                            // (rings of 2^12 points have no kernel that converts without the inverse pass: the rule must ask for it)
                            std::printf("decomposition: log_hi %u, digits of %u limbs, %u special primes, level %u, %u polynomials\n", log_hi, alpha, k, level, n);
                            return 1;
                        }
                    }
                    for (u32 merged = 0; merged <= (level ? 1 : 0); merged++) {
                        const u32 nd = k + merged, ap = merged ? k2_pad : k_pad;
                        if (!takes(log_hi, ap, nd, mid_conv_per(log_hi, nd, ap, level + 1 - merged, 2 * n))) {
                            std::printf("division: log_hi %u, %u special primes, level %u, %u ciphertexts, merged %u\n", log_hi, k, level, n, merged);
                            return 1;
                        }
                    }
                    if (level && !takes(log_hi, 4, 1, mid_conv_per(log_hi, 1, 4, level, 2 * n))) {
                        std::printf("rescale: log_hi %u, level %u, %u ciphertexts\n", log_hi, level, n);
                        return 1;
                    }
                }
            }
        }
    // refused: rings of 2^12 points without the inverse pass, rings that do not exist, more limbs than a row or a column holds
    for (u32 ap = 4; ap <= 16; ap += 4)
        for (u32 nd = 0; nd <= 17; nd++)
            for (u32 log_hi : {0u, 1u, 7u})
                if (hi_conv_terms(log_hi, ap, nd)) {
                    std::printf("a kernel for log_hi %u\n", log_hi);
                    return 1;
                }
    if (hi_conv_terms(4, 4, 5) || hi_conv_terms(4, 16, 17) || hi_conv_terms(4, 8, 0) || hi_conv_terms(4, 5, 5) || mid_conv_terms(1, 17) || mid_conv_terms(2, 11) ||
        mid_conv_terms(3, 6) || mid_conv_terms(4, 1) || mid_conv_terms(0, 1) || mid_conv_terms(1, 0) || conv_has_mid(4, 12, 10) || conv_has_mid(4, 12, 8)) {
        std::printf("a kernel for a size that has none\n");
        return 1;
    }
    // nothing is instantiated that no conversion reaches: the kernels of rows with their terms, and the columns
    for (u32 log_hi = 1; log_hi <= 6; log_hi++) {
        for (u32 ap = 4; ap <= 16; ap += 4)
            for (u32 nd = 1; nd <= ap; nd++)
                if (hi_conv_terms(log_hi, ap, nd) == nd && !reached.count({log_hi, ap, nd, false}) && !reached.count({log_hi, ap, nd, true})) {
                    std::printf("not reached: log_hi %u, rows of %u, %u terms\n", log_hi, ap, nd);
                    return 1;
                }
        for (u32 nd = 1; nd <= 16; nd++)
            if (mid_conv_terms(log_hi, nd) == nd && !reached.count({log_hi, 0u, nd, true})) {
                std::printf("not reached: log_hi %u, %u columns\n", log_hi, nd);
                return 1;
            }
    }
    std::fprintf(stderr, "%llu conversions\n", n_sizes);
    return 0;
}
