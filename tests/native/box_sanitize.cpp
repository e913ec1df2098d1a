// Sanitizer driver for the stencil boxes of the particle kernels
// (paper_1812_03689_amd/csrc/amrmg_box.hpp), built with
// -fsanitize=address,undefined by tests/test_sanitize_box.py: boxes from the
// minima that the kernels form, also those of wavefronts and workgroups
// without a particle inside the domain.
#include <cstdio>
#include <cstdlib>

#include "amrmg_box.hpp"

using namespace amrmg;

static void fail(const char *m)
{
    std::printf("box: %s\n", m);
    std::exit(1);
}

int main()
{
    CellBox B;
    const int none[6] = {INT_MAX, INT_MAX, INT_MAX, INT_MAX, INT_MAX, INT_MAX};
    B.set(none);
    if (!B.empty() || B.vol != 0 || B.nbt != 0) fail("no particle: not empty");
    const int lows[] = {0, 1, 7, 8, 63, 4088, 262136}, spans[] = {1, 2, 8, 9, 100};
    for (int lo : lows)
        for (int sx : spans)
            for (int sy : spans)
                for (int sz : spans) {
                    const int v[6] = {lo, lo + 3, lo + 5, ~(lo + sx - 1), ~(lo + 3 + sy - 1), ~(lo + 5 + sz - 1)};
                    B.set(v);
                    const int b[3] = {(lo + sx - 1) / 8 - lo / 8 + 1, (lo + 3 + sy - 1) / 8 - (lo + 3) / 8 + 1,
                                      (lo + 5 + sz - 1) / 8 - (lo + 5) / 8 + 1};
                    if (B.empty() || B.vol != (int64_t)sx * sy * sz || B.ex != sx || B.ey != sy || B.ez != sz)
                        fail("extents");
                    if (B.nbx != b[0] || B.nby != b[1] || B.nbt != b[0] * b[1] * b[2]) fail("bricks");
                }
    std::printf("box sanitize ok\n");
    return 0;
}
