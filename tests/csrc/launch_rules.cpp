// Prints the launch sizes of csrc/fpt_launch.h: one line per argument triple "rule count cus".
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "fpt_launch.h"

int main(int argc, char **argv) {
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
