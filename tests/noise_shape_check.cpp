// The split of the modified-equilibrium noise over blocks for every extent,
// both precisions and every batch of steps: the LDS its kernels ask for must
// hold their lines and be no more than a compute unit has.  Host only.  Prints the number of splits that
// do not fit and the first of them.

#include <cstdio>

#include "../paper_1012_3632_amd/csrc/internal.h"

int main() {
    long tried = 0, bad = 0;
    auto look = [&](int nx, int ny, int prec, int nb) {
        flb::ModEqArgs a{};
        a.nx = nx;
        a.ny = ny;
        a.prec = prec;
        const flb::ModEqNoiseShape s = flb::modeq_noise_shape(a, prec, nb);
        const size_t c = prec == 0 ? 8 : 16, cx = s.x64 ? 16 : c, cy = s.y64 ? 16 : c;
        // never less than the lines themselves
        const bool ok = s.NX >= 1 && s.NI >= 1 && s.NC >= 1 && s.lds_x <= flb::LDS_BYTES &&
                        s.lds_i <= flb::LDS_BYTES && s.lds_cols <= flb::LDS_BYTES &&
                        s.lds_x >= cx * (s.NX + 1) * nx && s.lds_i >= c * (s.NI + 1) * nx &&
                        s.lds_cols >= 2 * cy * s.NC * ny;
        ++tried;
        if (!ok && bad++ == 0)
            std::printf("first: %d x %d prec %d batch %d: rows %d, %zu and %d, %zu bytes; columns "
                        "%d, %zu bytes\n", nx, ny, prec, nb, s.NX, s.lds_x, s.NI, s.lds_i, s.NC,
                        s.lds_cols);
    };
    for (int prec = 0; prec < 2; ++prec) {
        for (int nx = 1; nx <= 1024; ++nx)
            for (int ny = 1; ny <= 1024; ++ny)
                for (int nb : {1, flb::MODEQ_MAX_BATCH}) look(nx, ny, prec, nb);
        // the other batches where a line's length and the lines there are of it
        // are far apart
        for (int n = 1; n <= 1024; ++n)
            for (int m : {1, 63, 126, 256, 512, 1024})
                for (int nb = 2; nb < flb::MODEQ_MAX_BATCH; ++nb) {
                    look(n, m, prec, nb);
                    look(m, n, prec, nb);
                }
    }
    std::printf("%ld splits, %ld do not fit\n", tried, bad);
    return bad != 0;
}
