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

static void few_inputs() {
    const Route C = Route::kColumns, B = Route::kBricks, S = Route::kSlabs;
    const char* const name[] = {"columns", "bricks", "slabs"};
    struct {
        Geo g;
        int ci, co;
        bool groups32;
        Route route;
    } at[] = {
        {{1, 300, 1, 79}, 32, 32, true, B},     // 11.2 us, by columns 13.8
        {{3, 14, 4, 295}, 32, 96, true, B},     // 19.0, 22.7
        {{2, 300, 3, 25}, 32, 96, true, B},     // 21.6, 25.0
        {{3, 30, 255, 3}, 32, 128, false, S},   // 50.9, 65.2
        {{20, 218, 10, 3}, 32, 64, false, S},   // 47.3, 84.0
        {{1, 100, 128, 128}, 32, 32, true, C},  // 78, by bricks 128
        {{4, 64, 32, 32}, 32, 96, true, C},     // 49, 84
        {{1, 100, 57, 57}, 32, 64, false, C},   // 56, from slabs 110
        {{3, 300, 3, 1}, 16, 96, true, B},      // 10.3, 14.6
        {{1, 172, 2, 149}, 16, 32, true, B},    // 8.8, 11.6
        {{4, 99, 4, 298}, 16, 64, true, B},     // 45.0, 55.0
        {{3, 16, 8, 253}, 16, 64, true, B},     // 11.9, 13.8
        {{3, 300, 73, 1}, 16, 128, false, S},   // 33.1, 95.6
        {{24, 61, 9, 6}, 16, 128, false, S},    // 34.8, 45.1
        {{1, 100, 128, 128}, 16, 32, true, C},  // 48, by bricks 74
    };
    for (const auto& a : at) {
        char what[90];
        const Route got = route_few(a.g, a.ci, a.co, a.groups32);
        std::snprintf(what, sizeof what, "%d -> %d, %d x %d x %d x %d: %s, %s wanted", a.ci, a.co,
                      a.g.B, a.g.D, a.g.H, a.g.W, name[(int)got], name[(int)a.route]);
        check(what, got == a.route);
    }
    // a batch of single voxels: more columns than a launch has workgroups
    check("10M volumes, 64 -> 64: by bricks", plan_wide({10000000, 1, 1, 1}, 64).planes == 0);
    check("10M volumes, 32 -> 64: from slabs", route_few({10000000, 1, 1, 1}, 32, 64, false) == S);
    check("10M volumes, 16 -> 96: by bricks", route_few({10000000, 1, 1, 1}, 16, 96, true) == B);
    // the split: every plane once, and no other split modelled as faster
    for (int D = 1; D <= 120; ++D)
        for (const long long cols : {1, 3, 64, 130, 257, 511, 513, 2000}) {
            const March m = plan_march(D, cols, 180, 160, 250);
            long long best = 1LL << 60;
            for (int n = 1; n <= D; ++n) {
                const long long it = cols * ceil_div(D, n);
                best = std::min(best, 180 + (n + 2) * (250 * ((it - 1) / 512) +
                                                       (last_round(it, 512) <= 256 ? 160 : 250)));
            }
            if (m.cost != best || m.items != cols * ceil_div(D, m.planes) || m.planes < 1 ||
                m.planes > D)
                check("a split into columns", false);
            if (D % 2 == 0) {
                const March e = plan_march(D, cols, 180, 160, 250, 2);
                if (e.planes % 2 || e.items != cols * ceil_div(D, e.planes))
                    check("a split into columns of even length", false);
            }
        }
}

static void sixteen() {
    struct {
        Geo g;
        int groups;
        bool columns;
    } at[] = {
        {{4, 300, 4, 255}, 3, false},    // by bricks 65 us, by columns 153
        {{25, 220, 8, 19}, 3, false},    // 62, 106
        {{27, 259, 19, 19}, 1, false},   // 62, 88
        {{2, 111, 89, 136}, 1, false},   // 46, 52
        {{1, 259, 119, 176}, 3, true},   // 775, 279
        {{4, 111, 59, 31}, 3, true},     // 59, 39
        {{1, 200, 256, 256}, 1, true},   // 235, 177
        {{4, 128, 64, 64}, 1, true},     // 36.0, 33.8
        {{1, 100, 40, 40}, 1, false},    // 8.2, 9.8
        {{1 << 25, 1, 1, 1}, 1, false},  // more columns than a launch has workgroups
        {{1 << 22, 1, 2, 2}, 1, false},
    };
    for (const auto& a : at) {
        char what[90];
        March m;
        const bool got = plan_march16(a.g, a.groups, 1, false, &m);
        std::snprintf(what, sizeof what, "16 -> %d, %d x %d x %d x %d: by %s", 16 * a.groups, a.g.B,
                      a.g.D, a.g.H, a.g.W, a.columns ? "columns" : "bricks");
        check(what, got == a.columns && (!got || m.items < (1 << 24)));
    }
    March m;   // pooled: 54 us by bricks, 45 by columns
    check("pooled 120 x 136 x 136: by columns", plan_march16({1, 120, 136, 136}, 1, 2, true, &m));
}

static void concatenation() {
    struct {
        Geo g;
        int planes;   // 0: by bricks
    } at[] = {
        {{1, 200, 192, 192}, 29},   // 143 us less than by bricks, 38 in columns of 200 planes
        {{1, 200, 200, 200}, 67},   // 180, 77
        {{1, 200, 264, 264}, 29},   // 285, 38
        {{1, 200, 256, 264}, 20},   // 222, 12
        {{1, 200, 256, 256}, 200},  // 289
        {{4, 128, 64, 64}, 32},     // 39
        {{1, 200, 72, 72}, 20},     // 15
        {{2, 100, 8, 200}, 0},      // 8 us more than by bricks
        {{4, 128, 16, 16}, 0},      // 2
        {{3, 50, 6, 90}, 0},        // 6
        {{1, 40, 80, 80}, 0},       // 1
        {{1, 64, 8, 8}, 0},         // 2
    };
    for (const auto& a : at) {
        char what[90];
        int n = 0;
        const bool got = plan_cat16(a.g, &n);
        std::snprintf(what, sizeof what, "concatenation %d x %d x %d x %d: %d planes, %d wanted", a.g.B,
                      a.g.D, a.g.H, a.g.W, got ? n : 0, a.planes);
        check(what, (got ? n : 0) == a.planes);
    }
}

static void weight_gradients() {
    struct {
        Geo g;
        int ci, co;
        bool slices;
    } at[] = {
        {{2, 300, 1, 1}, 16, 192, true},     // 14.3 us, by columns 31.3
        {{41, 50, 2, 4}, 128, 96, true},     // 91, 175
        {{16, 300, 1, 4}, 32, 48, true},     // 44, 51
        {{1, 300, 7, 1}, 16, 96, true},      // 16.4, 19.5
        {{1, 35, 38, 18}, 96, 96, false},    // 86, 38
        {{2, 300, 70, 2}, 32, 96, false},    // 192, 102
        {{2, 300, 1, 1}, 16, 64, false},     // bricks before: columns
    };
    for (const auto& a : at) {
        char what[90];
        const bool got = wgrad_by_slices(a.g, a.ci, a.co, wgrad_cols_plan(a.g, a.ci, a.co, 1000));
        std::snprintf(what, sizeof what, "weight gradient %d -> %d, %d x %d x %d x %d: %s", a.ci, a.co,
                      a.g.B, a.g.D, a.g.H, a.g.W, a.slices ? "slices" : "columns");
        check(what, got == a.slices);
    }
}

int main() {
    wide();
    weight_gradients();
    concatenation();
    few_inputs();
    sixteen();
    std::printf("done: %d failures\n", failures);
    return failures ? 1 : 0;
}
