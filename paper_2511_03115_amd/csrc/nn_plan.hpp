// Which kernel takes a convolution's layer, and how it is split: modelled
// times, in units of 10 ns, of launches on the 256 CUs of an MI355X.  Plain
// arithmetic on sizes, shared with a CPU build that checks it.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

namespace sde {
namespace nn {

struct Geo {
    int B, D, H, W;
    __host__ __device__ __forceinline__ long long nvox() const { return (long long)B * D * H * W; }
};

constexpr int kRZ = 4, kRY = 4, kRX = 16;   // the brick of the brick kernels

inline long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }
inline long long bricks_of(const Geo& g) {
    return ceil_div(g.W, kRX) * ceil_div(g.H, kRY) * ceil_div(g.D, kRZ) * g.B;
}
// columns of 16 x ry voxels
inline long long columns_of(const Geo& g, int ry) {
    return ceil_div(g.W, 16) * ceil_div(g.H, ry) * g.B;
}

// Workgroups beyond whole rounds of `round`: 1..round of them.
inline long long last_round(long long items, long long round) {
    return items - (items - 1) / round * round;
}

// ---- 64 and more inputs, groups of 32 outputs ------------------------------
// k_conv_wide in blocks of 1, 2 or 4 planes, or k_conv_fwd_pass by bricks
// (planes = 0); time per pass of 32 channels.
//
// Blocks take 3.0, 3.65 and 5.1 us for every 256 of them; bricks, two of which
// share a CU, 7.9 per 512 and 5.0 or 7.1 for what is left (fits to 400 random
// shapes; 4.7 us of start for either).  So blocks are the faster by half where
// they are full, and bricks where the volume has few rows or planes, or where
// the blocks are a few more than the CUs: 64 -> 64 on 4 x 63 x 3 x 73 voxels 33.6
// us by bricks and 36.9 by blocks of 4 planes, on 2 x 148 x 12 x 10 22.2 and 27.1;
// 96 -> 128 on 4 x 1 x 222 x 3 20.2 us in blocks of 1, 32.5 in blocks of 4;
// 100 x 128 x 128, 96 -> 32: 353 by bricks, 234 in blocks of 4.
struct WidePlan {
    int planes;
    long long cost;
};
inline WidePlan plan_wide(const Geo& g, int Co) {
    const long long cols = columns_of(g, 8) * (Co / 32), nb = bricks_of(g) * (Co / 32);
    WidePlan best{0, 790 * ((nb - 1) / 512) + (last_round(nb, 512) <= 256 ? 500 : 710)};
    const int planes[3] = {1, 2, 4}, time[3] = {300, 365, 510}, start[3] = {0, 0, 45};
    for (int k = 2; k >= 0; --k) {
        const long long c =
            time[k] * ceil_div(cols * ceil_div(g.D, planes[k]), 256) + start[k];
        if (c <= best.cost) best = WidePlan{planes[k], c};
    }
    return best;
}

}  // namespace nn
}  // namespace sde
