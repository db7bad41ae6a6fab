// Host check of tile_read (lbm_kernels.h): every address that the adjoint tile forms
// lies in a state of the caller's, or is past the end for the bounds check.
#include <cstdio>

#include "lbm_kernels.h"

int main() {
    using namespace lbm;
    // the largest state of a grid that goes by tiles: 256 strips x 48 rows x 48 columns
    const unsigned bytes = 9u * CHUNK * 8u * (unsigned)chunks_of((int64_t)256 * 48 * 48);
    for (int S = 1; S <= MAX_STEPS_PER_PASS; ++S)
        for (int j = 1; j <= S + 1; ++j)
            for (int owned = 0; owned < 2; ++owned) {
                const TileRead r = tile_read(j, S, owned != 0);
                const bool reads = j <= S && owned;
                if (r.step < 1 || r.step > S || (reads && r.step != j)) return 1;
                if (reads != (r.skip == 0)) return 2;
                for (int plane = 0; plane < 9; ++plane) {
                    const unsigned scalar = plane * (unsigned)CHUNK * 8u;
                    if (scalar >= bytes) return 3;  // size less scalar offset stays positive
                    for (unsigned off : {0u, bytes - 8u})
                        if (!reads && (off | r.skip) < bytes - scalar) return 4;
                }
            }
    std::puts("ok");
    return 0;
}
