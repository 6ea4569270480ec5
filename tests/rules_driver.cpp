// Prints what csrc/rules.h answers, one line per request on standard input:
//   finish K LONGEST  waves per tensor, tensors per workgroup of the norm's finish
//   pinned FLAGS      1 when the copy kernel may move memory allocated with these flags
#include <cstdio>
#include <iostream>
#include <string>

#include "rules.h"

int main()
{
    std::string what;
    while (std::cin >> what) {
        if (what == "finish") {
            int k;
            long long longest;
            std::cin >> k >> longest;
            const rules::FinishGeom g = rules::finish_geom(k, longest);
            std::printf("%d %d\n", g.waves, g.tensors);
        } else if (what == "pinned") {
            unsigned flags;
            std::cin >> flags;
            std::printf("%d\n", int(rules::copy_kernel_takes(flags)));
        } else {
            return 1;
        }
    }
    return 0;
}
