// Host check of where the backward pass of the fine-tuning loss looks for a token's teacher logits: with argument lists of M V r,
// the rows of the first chunk, and the first element of its last token's row, as "rows start".
#include <cstdio>
#include <cstdlib>
#include "tile_walk.hpp"

int main(int argc, char **argv)
{
    for (int i = 1; i + 2 < argc; i += 3) {
        const size_t M = std::strtoull(argv[i], nullptr, 10), V = std::strtoull(argv[i + 1], nullptr, 10), r = std::strtoull(argv[i + 2], nullptr, 10);
        const size_t rows = backward_chunk_rows(M, (V + 63) / 64 * 64, false) / r * r;
        std::printf("%zu %zu\n", rows, teacher_row_start((int)(rows / r - 1), (int)V));
    }
    return 0;
}
