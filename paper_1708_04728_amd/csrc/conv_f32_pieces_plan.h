// Which layers conv_f32_pieces.hip takes, with which tiles, and how the workgroups of a launch share the tiles of its layers.  Plain functions of numbers, so that
// the same lines run in the launcher and on the host.
#pragma once
#include <math.h>

namespace dr {

// Tiles of filters x pixels, and the most input pixels under one (LDS holds them twice)
constexpr int PIECES_TILES = 4;
// microseconds of a tile: fixed + slices * slice, fitted to 90 layers each (10, 8, 8 and 10 % off)
struct PiecesTile { int bm, bn, patch; double fixed, slice; };
constexpr PiecesTile pieces_tiles[PIECES_TILES] = {{128, 128, 512, 6.9, 0.92}, {96, 128, 512, 5.1, 0.79}, {64, 128, 512, 3.1, 0.64}, {64, 256, 640, 6.5, 0.90}};

struct PiecesLayer { int N, C, H, W, K, R, S, sh, sw, P, Q; };

// slices of 32 of the contraction, two filter taps of 16 channels each
constexpr int pieces_slices(const PiecesLayer& l) { return (l.R * l.S * (l.C / 16) + 1) / 2; }

// Whether a tile's patch fits: consecutive outputs span at most `rows` rows of the images that they touch, each image R - 1 more input rows; and the loading
// lanes take at most a unit of 256 / 2 pixels each slice, in the slices of a block of 16 channels but those that it shares with its neighbours.
constexpr bool pieces_fits(const PiecesLayer& l, const PiecesTile& t)
{
    const long PQ = (long)l.P * l.Q;
    const long rows = (t.bn - 2) / l.Q + 2 + ((t.bn - 2) / PQ + 2) * (l.R - 1), pixels = rows * (l.Q + l.S - 1);
    return pixels <= t.patch && pixels <= l.R * l.S / 2 * 128;
}

constexpr long pieces_count(const PiecesLayer& l, const PiecesTile& t)
{
    return ((long)l.K + t.bm - 1) / t.bm * (((long)l.N * l.P * l.Q + t.bn - 1) / t.bn);
}

constexpr double pieces_cost(const PiecesLayer& l, const PiecesTile& t) { return t.fixed + pieces_slices(l) * t.slice; }

// The fastest tile of a layer by itself; -1: none fits.  us: the time it takes
inline int pieces_best(const PiecesLayer& l, int cus, double* us)
{
    int best = -1;
    for (int i = 0; i < PIECES_TILES; ++i) {
        if (!pieces_fits(l, pieces_tiles[i])) continue;
        const double t = 3.0 + ceil((double)pieces_count(l, pieces_tiles[i]) / cus) * pieces_cost(l, pieces_tiles[i]);
        if (best < 0 || t < *us) { best = i; *us = t; }
    }
    return best;
}

// Whether a layer is faster so than in the other fp32 kernels.  Their times are fitted as well: layers of up to 5.5 blocks of 32 x 32 outputs per compute unit, which the
// small-layer kernel takes (6 % off), and larger ones in tiles of 64 x 64 or 32 x 128 (7 %).  Of 133 layers drawn around the line none is slower than before
// with the margin of a tenth, the choice takes 1.007 times the best one's time on average, and they gain a factor of 1.23; the line in figures: 3x3 96 -> 96 on
// 28 x 28 x 12 29.2 us there and 32.0 here, 32 -> 96 on 28 x 28 x 16 14.3 and 14.1, 160 -> 128 on 28 x 28 x 11 43.6 and 36.4, 32 -> 128 on 27 x 27 x 15 17.4 and 12.8;
// of 70 more, on rectified operands, one is slower (3x3 64 -> 40 on 18 x 68 x 119 91.2 and 94.3).
// Contractions of up to nine slices, whose tiles are mostly start and end, have a wider margin (3x3 16 -> 360 on 5 x 13 x 63 10.4 and 12.0, 32 -> 232 on 12 x 67 x 22 29.7 and 31.5); eight taps (2x4 16 -> 43
// on 21 x 21 x 75 9.1 and 10.6, 144 -> 69 on 32 x 25 x 12 27.7 and 30.5) stay there, and 32 filters use half of a tile here: 3x3 192 -> 32 on 68 x 70 x 30 196 and 238.
// Fewer tiles than three for four compute units leave room that the layers of a module's depth would fill in one launch of the other kernels: the fused form of 5a on 64
// images, with a 3x3 160 -> 320 of 125 tiles, 132 us there and 142 here, so they have a wider margin too.  Up to two blocks of 32 x 32 per compute unit the others are at
// least twice as fast (tiles here leave most compute units idle).
inline bool pieces_pays(const PiecesLayer& l, int cus)
{
    if (l.sh != 1 || l.sw != 1 || l.C % 16 != 0 || l.R * l.S < 9 || (long)l.P * l.Q > 65536 || (long)l.P + l.R > 65536) return false;
    const double Ng = (double)l.N * l.P * l.Q, slices = (double)l.R * l.S * (l.C / 16);
    const double small = ceil(Ng / 32) * ((l.K + 31) / 32) / cus;
    if (small <= 2) return false;
    double other = 5.1 + 0.20 * small + 0.100 * small * slices;
    if (small > 5.5) {
        const bool rows32 = (l.K + 31) / 32 * 32 < (l.K + 63) / 64 * 64;
        const double tiles = rows32 ? ((l.K + 31) / 32) * ceil(Ng / 128) / cus : ((l.K + 63) / 64) * ceil(Ng / 64) / cus;
        other = 5.6 + 0.61 * tiles + 0.277 * tiles * slices + 0.282 * (ceil(tiles) - tiles) * slices;
    }
    double us = 0;
    const int best = pieces_best(l, cus, &us);
    if (best < 0) return false;
    return us < (4 * pieces_count(l, pieces_tiles[best]) < 3 * cus ? 0.7 : pieces_slices(l) <= 9 ? 0.75 : 0.9) * other;
}

// How the workgroups share the tiles of up to 4 layers: for each layer ranges of workgroups with the same number of tiles each
constexpr int PIECES_RANGES = 10, PIECES_LAYERS = 4;      // (each layer splits at most one range into three)
struct PiecesShare { int n; int first[PIECES_RANGES + 1], per[PIECES_RANGES], tile[PIECES_RANGES]; };      // workgroups [first[i], first[i + 1]): per[i] tiles each, from tile[i] on
struct PiecesPlan { int workgroups; double us; PiecesShare layer[PIECES_LAYERS]; };

// Layers in the given order (the longest tiles first); each fills up the workgroups that have least to do
inline bool pieces_plan(int n, const long* tiles, const double* cost, int cus, PiecesPlan* plan)
{
    struct { int n; double load; } cls[PIECES_RANGES + 2] = {{cus, 0.0}};
    int classes = 1;
    for (int j = 0; j < n; ++j) {
        // the least time t in which the workgroups can take all the tiles: one of load + i * cost
        auto room = [&](double t) { long r = 0; for (int c = 0; c < classes; ++c) r += t > cls[c].load ? cls[c].n * (long)((t - cls[c].load) / cost[j] + 1e-6) : 0; return r; };
        double best = -1;
        for (int c = 0; c < classes; ++c) {
            long lo = 1, hi = tiles[j];
            if (room(cls[c].load + hi * cost[j]) < tiles[j]) continue;
            while (lo < hi) {
                const long mid = (lo + hi) / 2;
                if (room(cls[c].load + mid * cost[j]) >= tiles[j]) hi = mid; else lo = mid + 1;
            }
            if (best < 0 || cls[c].load + lo * cost[j] < best) best = cls[c].load + lo * cost[j];
        }
        if (best < 0) return false;
        PiecesShare& s = plan->layer[j];
        s.n = 0;
        long left = tiles[j];
        int wg = 0, out = 0;
        struct { int n; double load; } next[PIECES_RANGES + 2];
        for (int c = 0; c < classes; ++c) {
            const long per = best > cls[c].load ? (long)((best - cls[c].load) / cost[j] + 1e-6) : 0;
            int n_left = cls[c].n;
            while (n_left > 0) {                 // whole workgroups, then one with what is left, then those with nothing
                const long take = per < left ? per : left;
                const int m = take > 0 ? (int)(left / take < n_left ? left / take : n_left) : n_left;
                if (s.n == PIECES_RANGES || out == PIECES_RANGES + 1) return false;
                s.first[s.n] = wg; s.per[s.n] = (int)take; s.tile[s.n] = (int)(tiles[j] - left);
                ++s.n;
                next[out].n = m; next[out].load = cls[c].load + take * cost[j];
                ++out;
                wg += m; n_left -= m; left -= m * take;
            }
        }
        s.first[s.n] = wg;
        classes = out;
        for (int c = 0; c < out; ++c) { cls[c].n = next[c].n; cls[c].load = next[c].load; }
        plan->us = best;
    }
    plan->us = 0;
    for (int c = 0; c < classes; ++c) plan->us = cls[c].load > plan->us ? cls[c].load : plan->us;
    plan->workgroups = cus;
    while (classes > 1 && cls[classes - 1].load == 0.0) plan->workgroups -= cls[--classes].n;
    return true;
}

// The tiles of up to 4 layers, in the given order, that end first: all combinations of two layers, else each layer's own best
inline bool pieces_choose(int n, const PiecesLayer* layer, int cus, int* type, PiecesPlan* plan)
{
    int at[PIECES_LAYERS];
    bool found = false;
    auto attempt = [&]() {
        long tiles[PIECES_LAYERS];
        double cost[PIECES_LAYERS];
        for (int i = 0; i < n; ++i) {
            tiles[i] = pieces_count(layer[i], pieces_tiles[at[i]]);
            cost[i] = pieces_cost(layer[i], pieces_tiles[at[i]]);
        }
        PiecesPlan p;
        if (!pieces_plan(n, tiles, cost, cus, &p) || (found && p.us >= plan->us)) return;
        *plan = p;
        found = true;
        for (int i = 0; i < n; ++i) type[i] = at[i];
    };
    if (n <= 2) {
        for (at[0] = 0; at[0] < PIECES_TILES; ++at[0])
            for (at[1] = 0; at[1] < (n == 2 ? PIECES_TILES : 1); ++at[1])
                if (pieces_fits(layer[0], pieces_tiles[at[0]]) && (n == 1 || pieces_fits(layer[1], pieces_tiles[at[1]]))) attempt();
    } else {
        double us;
        for (int i = 0; i < n; ++i) at[i] = pieces_best(layer[i], cus, &us);
        attempt();
    }
    return found;
}

}  // namespace dr
