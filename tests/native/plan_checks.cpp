// Evaluates the rule that chooses between the 3D step kernels on sizes timed
// with both.  Each line: the grid, the mode, the streaming kernel's tile there,
// and the kernel that is faster (0: streaming, else the short kernel's planes
// per block).
#include <cstdio>

#include "../../paper_2311_05038_amd/csrc/fd_plan.hpp"

struct Case {
    int64_t nz, ny, nx;
    bool f32, adjoint;
    int64_t tx, ty;
    int zc;
    bool stream;
};

int main()
{
    const Case cases[] = {
        // few rows of y, many blocks: most of a 16-row tile lies past the grid
        {700, 1, 6000, true, false, 128, 8, 0, false},
        {100, 3, 4000, true, false, 128, 8, 0, false},
        {1500, 8, 300, true, false, 128, 8, 0, false},
        {400, 17, 1000, true, false, 128, 8, 0, false},
        {100, 24, 4000, true, false, 128, 8, 0, false},
        {100, 40, 4000, true, false, 128, 8, 0, false},
        {100, 49, 4000, true, false, 128, 8, 0, false},
        {1000, 1, 500, true, true, 128, 8, 0, false},
        {1000, 17, 500, true, true, 128, 8, 0, false},
        {3000, 6, 4000, true, true, 256, 8, 0, true},
        {2000, 33, 2000, true, true, 256, 8, 0, true},
        {1000, 1, 500, false, false, 128, 8, 0, false},
        {1000, 5, 500, false, false, 128, 8, 0, false},
        // the same few rows, one round of blocks
        {40, 1, 300, true, false, 128, 8, 2, false},
        {100, 8, 1000, true, true, 128, 8, 2, false},
        {100, 8, 1000, false, false, 128, 8, 2, false},
        {2000, 1, 64, true, false, 128, 8, 2, false},
        // tiles that fit
        {64, 64, 64, true, false, 128, 8, 2, false},
        {96, 120, 152, true, true, 128, 8, 2, false},
        {53, 259, 333, true, false, 128, 8, 2, false},
        {100, 65, 1000, true, false, 128, 8, 2, false},
        {201, 333, 289, true, false, 128, 8, 4, false},
        {256, 256, 256, true, false, 128, 8, 4, false},
        {48, 48, 48, false, false, 128, 8, 2, false},
        {96, 120, 152, false, false, 128, 8, 4, false},
        {201, 333, 289, false, false, 128, 8, 0, false},
        // beyond the cache: the width in 128-wide tiles against the pitch
        {1024, 1024, 64, true, false, 128, 8, 4, true},
        {2165, 2165, 64, true, false, 128, 8, 4, true},
        {487, 972, 192, true, false, 128, 8, 4, true},
        {1120, 279, 192, true, false, 128, 8, 4, true},
        {1519, 1519, 130, true, false, 128, 8, 0, true},
        {300, 300, 300, true, false, 128, 8, 4, true},
        {577, 577, 300, true, false, 128, 8, 0, true},
        {1080, 1080, 257, true, false, 128, 8, 0, true},
        {1500, 65, 300, true, false, 128, 8, 0, true},
        {384, 384, 384, true, false, 128, 8, 0, true},
        {384, 384, 384, true, true, 128, 8, 4, true},
        {512, 512, 512, true, false, 256, 8, 0, true},
        {512, 512, 512, true, true, 256, 8, 4, true},
    };
    int bad = 0;
    for (const Case &c : cases) {
        const int64_t px = (c.nx + 63) / 64 * 64;
        const fdk::ShortPlan p = fdk::short_plan(c.nz, c.ny, c.nx, px, c.f32, c.adjoint, c.tx, c.ty);
        if (p.zc != c.zc || (p.zc > 0 && p.stream != c.stream)) {
            std::printf("%lld x %lld x %lld f32 %d adjoint %d: %d planes, stream %d; expected %d, %d\n",
                        (long long)c.nz, (long long)c.ny, (long long)c.nx, c.f32, c.adjoint, p.zc, p.stream, c.zc,
                        c.stream);
            ++bad;
        }
    }
    if (!bad) std::puts("plan checks passed");
    return bad != 0;
}
