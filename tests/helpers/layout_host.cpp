// Host harness around the scorers' layout arithmetic (dev_common.hpp): reads commands from
// stdin, prints results.
//   bucket e b0 cw nb  -> bucket number
//   class nb           -> extents per class
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
        } else {
            return 2;
        }
    }
    return 0;
}
