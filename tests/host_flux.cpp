// Host build of the edge-flux form of the cell operator (cube_math.h, cell_flux).
// stdin: ncomp, U[8*ncomp], w[6]; stdout: the 8*ncomp corner contributions.
#include <cstdint>
#include <cstdio>

#include "cube_math.h"

using namespace agca;

template <int NC>
static int run() {
    double U[8][NC], w[6], F[8][NC];
    for (int k = 0; k < 8; ++k)
        for (int c = 0; c < NC; ++c)
            if (std::scanf("%lf", &U[k][c]) != 1) return 1;
    for (int s = 0; s < 6; ++s)
        if (std::scanf("%lf", &w[s]) != 1) return 1;
    cell_flux<NC, double>(U, w, F);
    for (int k = 0; k < 8; ++k)
        for (int c = 0; c < NC; ++c) std::printf("%.17g\n", F[k][c]);
    return 0;
}

int main() {
    int nc = 0;
    if (std::scanf("%d", &nc) != 1) return 1;
    return nc == 1 ? run<1>() : nc == 3 ? run<3>() : 1;
}
