// Prints what the plain path plans for a training step: T d V n r -> name=value pairs, tile edges and numbers of K-splits.
// The shapes of the products are those of the backward pass: {dY, dU} share a launch per chunk, {dH, dW, dG} one at the end.
#include <cstdio>
#include <cstdlib>

#include "f32_plan.hpp"

int main(int argc, char **argv)
{
    if (argc != 6) return 2;
    const long T = std::atol(argv[1]), d = std::atol(argv[2]), V = std::atol(argv[3]), n = std::atol(argv[4]), r = std::atol(argv[5]);
    const long M = T * n * r, nrd = n * r * d, row = (V + 3) / 4 * 4;
    long rows = (1L << 27) / row / r * r;            // 512 MiB of logit gradients at a time
    if (rows < r) rows = r;
    if (rows > M) rows = M;
    const cph::F32Plan z = cph::f32_plan(rows, V, d, false);
    const cph::F32Shape chunk[2] = {{rows, d, V}, {V, d, rows}}, weights[3] = {{T, d, nrd}, {nrd, d, T}, {r, d, T}};
    cph::F32Plan c[2], w[3];
    cph::f32_plan(chunk, 2, true, c);
    cph::f32_plan(weights, 3, true, w);
    std::printf("chunks=%ld z=%d chunk=%d dY=%d dU=%d weights=%d dH=%d dW=%d dG=%d\n", (M + rows - 1) / rows, cph::f32_tile_edge(z.kind),
                cph::f32_tile_edge(c[0].kind), c[0].splits, c[1].splits, cph::f32_tile_edge(w[0].kind), w[0].splits, w[1].splits, w[2].splits);
    return 0;
}
