// Host harness around the scorers' layout arithmetic (dev_common.hpp): reads commands from
// stdin, prints results.
//   bucket e b0 cw nb  -> bucket number
//   class nb           -> extents per class
//   period Dt          -> columns between two seeds of the lazy rows
//   lazy Dt f0 f1 f2 R -> Dt + 1 rows of the lazy walk seeded every R columns from the exact one
//   exact Dt f0 f1 f2 k0 -> Dt + 1 rows of the exact walk started at k0 <= 0
#include <cmath>
#include <cstdio>
#include <cstring>

#include "dev_common.hpp"

using namespace stt;

int main()
{
    char cmd[16];
    while (std::scanf("%15s", cmd) == 1) {
        unsigned a, b, c, d;
        if (!std::strcmp(cmd, "bucket")) {
            if (std::scanf("%u %u %u %u", &a, &b, &c, &d) != 4) return 2;
            std::printf("%u\n", bucket_number(a, b, c, d));
        } else if (!std::strcmp(cmd, "class")) {
            if (std::scanf("%u", &a) != 1) return 2;
            std::printf("%u\n", bucket_class(a));
        } else if (!std::strcmp(cmd, "period")) {
            if (std::scanf("%u", &a) != 1) return 2;
            std::printf("%d\n", lazy_period((int32_t)a));
        } else if (!std::strcmp(cmd, "lazy") || !std::strcmp(cmd, "exact")) {
            int e;
            const bool lazy = cmd[0] == 'l';
            if (std::scanf("%u %u %u %u %d", &a, &b, &c, &d, &e) != 5) return 2;
            const Trk t{0, (int32_t)a, b, c, d, 0};
            DdaF st = ddaf_init_at(t, lazy ? 0 : e);
            double Y = 0.0;
            for (int k = lazy ? 0 : e; k <= (int)a; ++k) {
                if (lazy) {
                    if (k % e == 0) Y = lazy_seed(st.num, st.invq);
                    std::printf("%u ", lazy_row(Y) - kRowHi);
                    Y = lazy_step(Y, st.del, st.invq);
                } else if (k >= 0) {
                    std::printf("%u ", exact_row(st.num, st.invq) - kRowHi);
                }
                ddaf_step(st);
            }
            std::printf("\n");
        } else {
            return 2;
        }
    }
    return 0;
}
