// Prints what csrc/rules.h answers, one line per request on standard input:
//   pinned FLAGS      1 when the copy kernel may move memory allocated with these flags
#include <cstdio>
#include <iostream>
#include <string>

#include "rules.h"

int main()
{
    std::string what;
    while (std::cin >> what) {
        if (what == "pinned") {
            unsigned flags;
            std::cin >> flags;
            std::printf("%d\n", int(rules::copy_kernel_takes(flags)));
        } else {
            return 1;
        }
    }
    return 0;
}
