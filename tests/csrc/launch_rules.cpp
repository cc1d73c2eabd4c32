// Prints the launch sizes of csrc/fpt_launch.h: one line per argument triple "rule count cus".  With "pieces
// n", reads offsets from standard input and prints the ends of the evaluation's pieces of at most n records
// and, last, the capacity they need.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "fpt_launch.h"

int main(int argc, char **argv) {
    if (argc == 3 && !std::strcmp(argv[1], "pieces")) {
        const uint64_t piece = std::strtoull(argv[2], nullptr, 10);
        std::vector<uint64_t> off;
        for (unsigned long long v; std::scanf("%llu", &v) == 1;) off.push_back(v);
        const int64_t n = static_cast<int64_t>(off.size()) - 1;
        for (int64_t i = 0; i < n;) {
            i = fpt::eval_piece_end(off.data(), n, i, piece);
            std::printf("%lld\n", static_cast<long long>(i));
        }
        std::printf("%llu\n", static_cast<unsigned long long>(fpt::eval_capacity(off.data(), n, piece)));
        return 0;
    }
    for (int i = 1; i + 2 < argc; i += 3) {
        const uint64_t n = std::strtoull(argv[i + 1], nullptr, 10);
        const int cus = std::atoi(argv[i + 2]);
        uint32_t v = 0;
        if (!std::strcmp(argv[i], "slots")) v = fpt::record_slots(n, cus);
        else if (!std::strcmp(argv[i], "waves")) v = fpt::record_waves_per_group(n, cus);
        else if (!std::strcmp(argv[i], "eval")) v = fpt::eval_groups(n, cus);
        else if (!std::strcmp(argv[i], "check")) v = fpt::check_groups(n, cus);
        else return 2;
        std::printf("%u\n", v);
    }
    return 0;
}
