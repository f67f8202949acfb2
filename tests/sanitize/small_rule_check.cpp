// Prints, for every "n p entries" on stdin, whether its search is made in one
// launch, and the bytes of LDS that takes; checks that the parts of that state
// follow one another without overlap.
#include <cstdio>

#include "small_rule.hpp"

int main() {
    long long n, p, nnz;
    while (std::scanf("%lld %lld %lld", &n, &p, &nnz) == 3) {
        const bool one = csbfs::small_fits(n, p, nnz);
        long long bytes = 0;
        if (one) {
            const csbfs::SmallLds l = csbfs::small_lds(n, p);
            const long long words = n / 64, R = n / p;
            const long long at[] = {l.pi, l.nb, l.view, l.buf, l.par, l.queue, l.total};
            const long long size[] = {words, 2 * words, p * words, (long long)l.nbuf * l.buf_words, (n + 1) / 2,
                                      2 * csbfs::kSmallQueue};
            for (int k = 0; k < 6; ++k)
                if (at[k] + size[k] > at[k + 1]) return 1;
            if (l.pi != 0 || l.buf_words < R / 64 + 1 + R / 63 + 1) return 1;
            bytes = 8LL * l.total;
        }
        std::printf("%d %lld\n", one ? 1 : 0, bytes);
    }
    return 0;
}
