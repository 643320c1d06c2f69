// Which tile and how many workgroups each layer gets where several share a launch of conv_bf16_wide.hip.  Plain C++, so that the same lines run in the
// launcher and in a test on the host.
#pragma once
#include <algorithm>

namespace dr {

// Blocks of 32 filters and of 32 pixels of a tile; a layer by itself takes one of the first ten, beside others their share of the device may ask for
// smaller ones
constexpr int WIDE_TILES[][2] = {{5, 7}, {4, 7}, {7, 4}, {6, 5}, {3, 7}, {6, 4}, {4, 4}, {2, 7}, {2, 5}, {4, 3}, {3, 4}, {2, 3}, {1, 7}, {1, 4}};
constexpr int WIDE_TILE_COUNT = sizeof(WIDE_TILES) / sizeof(WIDE_TILES[0]), WIDE_ALONE = 10;

// A tile's time: a slice takes its matrix work or its loads, whichever is longer, a tile 0.54 us and its store besides.  Fitted to 14 tiles on 60 layers.
inline float wide_tile_us(int tm, int tn, int slices)
{
    const float mn = (float)(tm * tn * 1024);
    return slices * std::max(0.644f * mn / 32768.f, 12.85f * (tm + tn) / 256.f) + 0.54f + 1.2f * mn / 10000.f;
}

constexpr int WIDE_LAYERS = 4;                           // most layers of a launch
constexpr float WIDE_POOL_US = 2.2f;                     // a group of items of the pooling layer beside them
struct WideLayer { int K, Ng, slices; };
struct WidePlan { int tile[WIDE_LAYERS], gn[WIDE_LAYERS], pool_share; };      // tile and workgroups per filter block of each layer; workgroups that pool

// Every layer's tile and workgroups so that the slowest layer is done as soon as possible: the shortest time T, by halving (to 1/256 of where it starts:
// closer than the model is), at which the layers' least numbers of workgroups -- rounds of each tile that fit T -- add up to at most the compute units.
// What is added to T by a launch is 2.5 to 4.5 us (kernel trace of 112 modules).  About 1 us on the host for three layers.
// pool_blocks: groups of items of a pooling layer beside them (0: none).
// False, and no plan, where the compute units do not suffice at any T: a layer takes at least a workgroup for each block of 224 filters (its tallest tile),
// and every layer and the pooling step whole eights of workgroups.
inline bool wide_plan(const WideLayer* layers, int n, int pool_blocks, int cus, WidePlan* plan)
{
    struct Option { int grid_m, grid_n; float us; } opt[WIDE_LAYERS][WIDE_TILE_COUNT];
    float lo = 0.f, hi = 0.f;
    long fewest = pool_blocks ? 8 : 0;
    for (int i = 0; i < n; ++i) {
        const WideLayer& l = layers[i];
        float least = 1e30f, longest = 0.f;
        int rows = l.K;
        for (int t = 0; t < WIDE_TILE_COUNT; ++t) {
            const int bm = WIDE_TILES[t][0] * 32, bn = WIDE_TILES[t][1] * 32;
            Option& o = opt[i][t];
            o = Option{(l.K + bm - 1) / bm, (l.Ng + bn - 1) / bn, wide_tile_us(WIDE_TILES[t][0], WIDE_TILES[t][1], l.slices)};
            least = std::min(least, o.us * o.grid_m * o.grid_n);
            longest = std::max(longest, o.us);
            rows = std::min(rows, o.grid_m);
        }
        lo += least / cus;
        hi += 2.f * least / cus + longest;
        fewest += (rows + 7) / 8 * 8;
    }
    if (fewest > cus) return false;
    lo += WIDE_POOL_US * pool_blocks / cus;
    hi += 2.f * WIDE_POOL_US * pool_blocks / cus + WIDE_POOL_US;
    auto fits = [&](float T) {
        int sum = 0;
        WidePlan p{};
        if (pool_blocks) {
            if (T < WIDE_POOL_US) return false;
            const int rounds = T >= WIDE_POOL_US * pool_blocks ? pool_blocks : (int)(T / WIDE_POOL_US);
            p.pool_share = sum = ((pool_blocks + rounds - 1) / rounds + 7) / 8 * 8;
        }
        for (int i = 0; i < n; ++i) {
            int best = cus + 1;
            for (int t = 0; t < WIDE_TILE_COUNT; ++t) {
                const Option& o = opt[i][t];
                if (o.us > T) continue;
                const int rounds = T >= o.us * o.grid_n ? o.grid_n : (int)(T / o.us), w = (o.grid_n + rounds - 1) / rounds, blocks = (w * o.grid_m + 7) / 8 * 8;
                if (blocks < best) { best = blocks; p.tile[i] = t; p.gn[i] = w; }
            }
            sum += best;
            if (sum > cus) return false;
        }
        *plan = p;
        return true;
    };
    while (!fits(hi)) hi *= 2.f;                         // (ends: every layer's rounds reach its tiles, one workgroup per filter block)
    for (int k = 0; k < 8; ++k) {
        const float T = 0.5f * (lo + hi);
        (fits(T) ? hi : lo) = T;
    }
    return true;
}

}  // namespace dr
