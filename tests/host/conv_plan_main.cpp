// The rules by which the denoiser's convolutions choose a kernel and its split
// (paper_2511_03115_amd/csrc/nn_plan.hpp), on the CPU: at sizes where both
// sides were measured the faster one is taken.  Exits non-zero when a check
// fails.
#include <cstdio>

#include "nn_plan.hpp"

using namespace sde::nn;

static int failures = 0;

static void check(const char* what, bool ok) {
    if (!ok) ++failures;
    std::printf("%-70s %s\n", what, ok ? "ok" : "FAILED");
}

static void wide() {
    struct {
        Geo g;
        int co, planes;   // 0: by bricks
    } at[] = {
        {{4, 1, 222, 3}, 128, 1},    // 96 inputs: 20.2 us, in blocks of 4 32.5
        {{48, 1, 18, 13}, 64, 1},    // 192: 43.6, 64.8
        {{1, 300, 1, 3}, 192, 0},    // 64: 20.0, in blocks of 4 26.0
        {{2, 148, 12, 10}, 64, 0},   // 64: 22.2, 27.1
        {{1, 50, 34, 17}, 64, 0},    // 128: 34.9, 47.8
        {{3, 195, 2, 123}, 96, 0},   // 192: 309, 435
        {{1, 100, 128, 128}, 32, 4}, // 96: 234, by bricks 353
        {{1, 50, 64, 64}, 64, 4},    // 192: 148, 191
        {{4, 32, 16, 16}, 64, 2},    // 64: 14.5, in blocks of 4 18.7, of 1 19.4
        {{4, 16, 8, 8}, 128, 1},     // 128: 17.2, 27.8, of 2 20.5
    };
    for (const auto& a : at) {
        char what[80];
        const int got = plan_wide(a.g, a.co).planes;
        std::snprintf(what, sizeof what, "wide %d x %d x %d x %d -> %d: %d planes, %d wanted", a.g.B,
                      a.g.D, a.g.H, a.g.W, a.co, got, a.planes);
        check(what, got == a.planes);
    }
}

int main() {
    wide();
    std::printf("done: %d failures\n", failures);
    return failures ? 1 : 0;
}
