// Reads lines "fits k N" (whether the FP64 matrix form takes that population) and
// "pays k n N move" (whether it pays at those sizes), "column q N k" (the particle and component of thread q of its proposals), and
// "lds slices nchunks kd moves" (LDS bytes of a 1-D move's workgroup, of several moves'
// and the moves whose random numbers that one holds).
#include <cstdio>
#include <cstring>

#include "gmm_common.hpp"
#include "internal.hpp"

int main() {
    char what[16];
    while (std::scanf("%15s", what) == 1) {
        long long a, b;
        unsigned q;
        int k, p = -1, i = -1;
        if (std::strcmp(what, "fits") == 0 && std::scanf("%d %lld", &k, &a) == 2) {
            std::printf("%d\n", smc::dd64_fits(k, a) ? 1 : 0);
        } else if (std::strcmp(what, "pays") == 0 && std::scanf("%d %lld %lld %d", &k, &a, &b, &p) == 4) {
            std::printf("%d\n", smc::dd64_pays(k, a, b, p != 0) ? 1 : 0);
        } else if (std::strcmp(what, "lds") == 0 && std::scanf("%d %d %d %lld", &p, &i, &k, &a) == 4) {
            const int batch = smc::multi_batch(k, p, true, static_cast<int>(a), false);
            std::printf("%zu %zu %d\n", smc::rwmh_dyn_lds_bytes(p, i, true, k),
                        smc::multi_dyn_lds_bytes(p, i, true, k, batch), batch);
        } else if (std::scanf("%u %lld %d", &q, &b, &k) == 3) {
            const bool in = smc::dd_column(q, static_cast<int>(b), k, p, i);
            std::printf("%d %d %d\n", in ? 1 : 0, p, i);
        }
    }
    return 0;
}
