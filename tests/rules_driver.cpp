// Prints what csrc/rules.h answers, one line per request on standard input:
//   finish K LONGEST  waves per tensor, tensors per workgroup of the norm's finish
//   percu B MAP N...  workgroups per CU of the 8-bit step (0: as many as fit) over tensors
//                     of N elements, without and with fp32 gradients or a bf16 copy; NxK
//                     stands for K tensors of N elements
//   percu32 N         workgroups per CU of the fp32-state step over N elements
//   geom B MAP N...   waves, granules and blocks per unit of k_adamw8_any (waves 0:
//                     k_adamw8_generic) for a block size that is no power of two
//   pinned FLAGS      1 when the copy kernel may move memory allocated with these flags
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "rules.h"

// The list of a request's remaining words: B, map, sizes (N or NxK).
static rules::StepList list_of(std::istringstream& in, std::vector<int64_t>& sizes)
{
    int B, map;
    in >> B >> map;
    std::string word;
    while (in >> word) {
        const size_t x = word.find('x');
        const long long n = std::stoll(word.substr(0, x));
        const long long k = x == std::string::npos ? 1 : std::stoll(word.substr(x + 1));
        sizes.insert(sizes.end(), size_t(k), int64_t(n));
    }
    return rules::step_list(sizes.data(), int(sizes.size()), B, map != 0);
}

int main()
{
    std::string line, what;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        in >> what;
        std::vector<int64_t> sizes;
        if (what == "finish") {
            int k;
            long long longest;
            in >> k >> longest;
            const rules::FinishGeom g = rules::finish_geom(k, longest);
            std::printf("%d %d\n", g.waves, g.tensors);
        } else if (what == "percu") {
            const rules::StepList l = list_of(in, sizes);
            std::printf("%d %d\n", rules::step_per_cu(l, false), rules::step_per_cu(l, true));
        } else if (what == "percu32") {
            long long n;
            in >> n;
            std::printf("%d\n", rules::step32_per_cu(n));
        } else if (what == "geom") {
            const rules::AnyGeom g = rules::any_geom(list_of(in, sizes));
            std::printf("%d %d %d\n", g.waves, g.granules, g.blocks);
        } else if (what == "pinned") {
            unsigned flags;
            in >> flags;
            std::printf("%d\n", int(rules::copy_kernel_takes(flags)));
        } else {
            return 1;
        }
    }
    return 0;
}
