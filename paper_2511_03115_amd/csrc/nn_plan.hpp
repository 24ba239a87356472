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

// a launch is below 2^32 threads, 256 to a workgroup
constexpr long long kMaxItems = (1LL << 24) - 1;

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
        const long long items = cols * ceil_div(g.D, planes[k]);
        const long long c = time[k] * ceil_div(items, 256) + start[k];
        if (c <= best.cost && items <= kMaxItems) best = WidePlan{planes[k], c};
    }
    return best;
}

// ---- columns that march along z --------------------------------------------
// n output planes each (a multiple of `multiple`, which divides D), one or two
// workgroups to a CU: base + (n + 2) x shared for every 512 of them and
// (n + 2) x alone or shared for what is left; without end where no split is few
// enough for a launch (32 -> 32, 4 x 64 x 32 x 32 voxels:
// n = 8, 256 workgroups 20.2 us, n = 6, 352: 24.3, n = 4, 512: 20.9; 2 x 50 x 24 x
// 40: n = 4, 234 workgroups 12.7, n = 2, 450: 13.9).
struct March {
    int planes;
    long long items, cost;
};
inline March plan_march(int D, long long cols, int base, int alone, int shared, int multiple = 1) {
    March best{D, cols, 1LL << 60};
    const int U = D / multiple;
    for (int u = U; u >= 1; --u) {
        const int k = (int)ceil_div(U, u);
        u = (int)ceil_div(U, k);   // the shortest columns of as many pieces
        const long long items = cols * k;
        const long long cost = base + (u * multiple + 2LL) * (shared * ((items - 1) / 512) +
                                                              (last_round(items, 512) <= 256 ? alone : shared));
        if (cost <= best.cost && items <= kMaxItems) best = March{u * multiple, items, cost};
    }
    return best;
}

// ---- 16 and 32 inputs, groups of 32 outputs --------------------------------
// By columns (k_conv_march, k_conv_march_pairs), by bricks (k_conv_fwd_reg), or,
// where the outputs are not taken 32 at a time, from weight slabs
// (k_conv_fwd_lds).  Fits to 2 x 400 random shapes: 16 inputs 3.3 us + (n + 2) 1.05
// alone, 1.55 shared; bricks 2.2 + 7.8 for every 768, 5.0, 6.8 or 8.6 for those
// left; slabs 0.19 ns per voxel and 64 outputs, 14.4 at least.  32 inputs 1.8 +
// (n + 2) 1.6 or 2.5; bricks 2.0 + 9.7 for every 512, 7.3 or 9.8; slabs 8 + 0.29
// ns, 21.3 at least.  Columns are twice as fast where they are full (100 x 128 x
// 128, 32 -> 32: 128 us by bricks, 78; 16 -> 32: 74 and 48); on volumes of one to
// four rows, or narrower than a column, they are not (32 -> 32 on 300 x 1 x 79: 11.2
// by bricks, 13.8; 16 -> 128 on 3 x 300 x 73 x 1: 33 from slabs, 96).
enum class Route { kColumns, kBricks, kSlabs };
inline March plan_columns(const Geo& g, int Ci, int Co) {
    const long long cols = columns_of(g, 8) * (Co / 32);
    return Ci == 16 ? plan_march(g.D, cols, 330, 105, 155) : plan_march(g.D, cols, 180, 160, 250);
}
inline Route route_few(const Geo& g, int Ci, int Co, bool groups32) {
    const long long columns = plan_columns(g, Ci, Co).cost;
    if (!groups32) {
        const long long v = g.nvox() * Co / 64;
        const long long slabs = Ci == 16 ? std::max(1440LL, 800 + v * 19 / 1000)
                                         : std::max(2130LL, 800 + v * 29 / 1000);
        return columns <= slabs ? Route::kColumns : Route::kSlabs;
    }
    const long long nb = bricks_of(g) * (Co / 32);
    long long bricks;
    if (Ci == 16) {
        const long long l = last_round(nb, 768);
        bricks = 220 + 780 * ((nb - 1) / 768) + (l <= 256 ? 500 : l <= 512 ? 680 : 860);
    } else {
        bricks = 200 + 970 * ((nb - 1) / 512) + (last_round(nb, 512) <= 256 ? 730 : 980);
    }
    return columns <= bricks ? Route::kColumns : Route::kBricks;
}

// ---- 16 inputs, 1 to 3 groups of 16 outputs ---------------------------------
// k_conv_march16's columns of 16 x 16 voxels, from 2M voxels and groups on (the
// persistent bricks of k_conv_rows have the shorter start: 100 x 40 x 40 voxels
// 8.2 us, columns 9.8; 1.6M: 30.2 and 31.7; 2.1M: 36.0 and 33.8; 13.1M: 235 and
// 177) and where their modelled time is the less by 6 %: 4.1 ns per brick, three
// groups 3.3 ps per voxel and group more, against (n + 2) planes of 1.01 or 1.62 us
// (fits to 2 x 450 random shapes).  On few rows most of a column lies beside the
// volume: 16 -> 48 on 4 x 300 x 4 x 255 65 us by bricks, 153 by columns; 16 -> 16 on 2
// x 111 x 89 x 136 46 and 52.  Columns add the 2 x 2 x 2 sums of their planes in
// registers and read the activations of a gradient ahead: with such outputs (fused)
// they may be modelled 8 % the slower (pooled, 120 x 136 x 136: 54 us by bricks, 45;
// a training step of 2 x 200 x 50 x 120 17 us less by columns).
inline bool plan_march16(const Geo& g, int groups, int multiple, bool fused, March* m) {
    const long long v = g.nvox() * groups;
    if (v < 1LL << 21) return false;
    *m = plan_march(g.D, columns_of(g, 16) * groups, 300, 101, 162, multiple);
    const long long rows = 300 + bricks_of(g) * groups * 41 / 100 + (groups > 2 ? v * 33 / 100000 : 0);
    return m->cost < 1LL << 40 && m->cost * (fused ? 92 : 106) < rows * 100;
}

// ---- the decoder's level-0 concatenation, 16 + 32 -> 16 ---------------------
// k_conv_cat16's columns of 16 x 16 voxels, one workgroup to a CU: as many planes
// each as make ceil(workgroups / 256) (n + 2), its time in units of 2.0 us, the
// least; where that, with 3 us, is less than 3.5 us for every 256 bricks of the
// persistent k_conv_rows.  As many columns' pieces as CUs, without a look at
// the rest, left them idle (differences to the bricks' whole forward pass: 192 x
// 192 x 200 voxels, 144 columns, -38 us in columns of 200 planes, -143 of 29; 264 x
// 264 x 200, 289 columns, -38 and -285; 256 x 256 x 200, of 200, -290), and small
// volumes are faster by bricks (2 x 100 x 8 x 200: +8 us by columns, 4 x 128 x 16 x 16
// +2, 80 x 80 x 40 +1; 72 x 72 x 200 -15).
inline bool plan_cat16(const Geo& g, int* planes) {
    const long long cols = columns_of(g, 16);
    long long best = 1LL << 60;
    for (int n = g.D; n >= 1; --n) {
        const int k = (int)ceil_div(g.D, n);
        n = (int)ceil_div(g.D, k);
        const long long c = ceil_div(cols * k, 256) * (n + 2);
        if (c <= best) {
            best = c;
            *planes = n;
        }
    }
    return 200 * best + 300 < 350 * ceil_div(bricks_of(g), 256);
}

// ---- weight gradients -------------------------------------------------------
// The split of k_wgrad_cols: n planes per column, ncol columns, cpw pairs of
// columns per half workgroup, used workgroups per channel block.
constexpr int kWgColsR = 2;
struct WgradCols {
    int n, ncol, cpw, used;
};
inline WgradCols wgrad_cols_plan(const Geo& g, int Ci, int Co, long long max_used) {
    const long long nxy = columns_of(g, 4 * kWgColsR);
    // one workgroup per CU in all, as far as the partial sums' buffer goes
    const long long want =
        std::max(1LL, std::min(max_used, 256LL / std::max(1, (Ci / 16) * (Co / 16))));
    // the plane count whose longest workgroup marches over the fewest planes
    // (of equals the longest columns)
    WgradCols p{};
    long long best = 1LL << 60;
    for (int nz = 1; nz <= std::min(g.D, 64); ++nz) {
        const int n = (int)ceil_div(g.D, nz);
        const long long ncol = nxy * ceil_div(g.D, n), pairs = (ncol + 1) / 2;
        const long long cpw = ceil_div(pairs, 2 * want);
        if (ncol > (1 << 29) || cpw * (n + 2) >= best) continue;
        best = cpw * (n + 2);
        p = WgradCols{n, (int)ncol, (int)cpw, (int)ceil_div(pairs, 2 * cpw)};
    }
    return p;
}

// Output widths other than 16, 32, 64 and 128 (which have never gone by them)
// take k_wgrad_partial's 64-voxel slices where a column is mostly beside the
// volume: columns 10.0 us, 1.3 for each plane a workgroup marches over and their
// partial sums' bytes at 2 TB/s there and back; slices 14 us + 0.22 ns, or 30 + 0.085,
// per voxel and channel block (fits to 2 x 100 random shapes; 16 -> 192 on 2 x 300 x 1
// x 1 31 us by columns, 14 from slices; 128 -> 96 on 41 x 50 x 2 x 4 175 and 91; 96 -> 96
// on 1 x 35 x 38 x 18 38 and 86).
inline bool wgrad_by_slices(const Geo& g, int Ci, int Co, const WgradCols& p) {
    if (Co == 16 || Co == 32 || Co == 64 || Co == 128) return false;
    const long long v = g.nvox() * (Ci / 16) * (Co / 16);
    const long long columns = 1000 + 130LL * p.cpw * (p.n + 2) + p.used * 27LL * Ci * Co / 5000;
    return std::min(1400 + v * 22 / 1000, 3000 + v * 85 / 10000) < columns;
}

}  // namespace nn
}  // namespace sde
