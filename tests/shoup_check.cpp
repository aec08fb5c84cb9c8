// Compares the lazy Shoup product with 128-bit integers: result below 4q and congruent to a * w, for random and extreme operands.
#include <cstdio>
#include "../paper_2604_16834_amd/csrc/shoup.h"

typedef unsigned __int128 u128;

static uint64_t state = 88172645463325252ull;
static uint64_t rnd() {
    state ^= state << 13;
    state ^= state >> 7;
    return state ^= state << 17;
}

int main() {
    const uint64_t qs[] = {(1ull << 58) - 27, (1ull << 58) - 1, (1ull << 57) + 1, (1ull << 56) - 5, 1152921504606846975ull >> 3, 12289, 3};
    unsigned long long worst = 0, n = 0;
    for (uint64_t q : qs) {
        const uint64_t nq = 0 - q;
        for (int i = 0; i < 400000; i++) {
            const uint64_t ws[] = {0, 1, q - 1, q / 2, rnd() % q}, as[] = {0, 1, ~0ull, ~0ull << 32, 0xffffffffull, q - 1, 60 * q, rnd(), rnd() >> 32, rnd() << 32};
            const uint64_t w = ws[i % 5], a = i < 4000 ? as[(i / 5) % 10] : rnd();
            const uint64_t w_sh = (uint64_t)(((u128)w << 64) / q), r = mul_shoup_lazy4(a, w, w_sh, nq);
            if (r >= 4 * q || (uint64_t)((u128)a * w % q) != r % q) {
                std::printf("q %llu a %llu w %llu: %llu\n", (unsigned long long)q, (unsigned long long)a, (unsigned long long)w, (unsigned long long)r);
                return 1;
            }
            if (r / q > worst) worst = r / q;
            n++;
        }
    }
    std::printf("%llu products, largest quotient error %llu\n", n, worst);
    return 0;
}
