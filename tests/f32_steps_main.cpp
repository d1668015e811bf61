// Prints the K-step of a launch of 128-wide tiles with two K-contiguous operands: argument lists of tiles, bfloat16 operands, 0 or 1
// for four elements per load.
#include <cstdio>
#include <cstdlib>

#include "f32_plan.hpp"

int main(int argc, char **argv)
{
    for (int i = 1; i + 2 < argc; i += 3)
        std::printf("%d\n", cph::f32_short_steps(std::atol(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2]) != 0) ? 16 : 32);
    return 0;
}
