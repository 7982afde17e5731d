// Tile / schedule choice of the stage kernel per (precision, dimension, size).
// Defaults are set here; ofm_tune_set overrides one entry and ofm_autotune
// measures the compiled candidates and stores the fastest unless what is used
// without it is faster.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <map>
#include <tuple>

namespace ofm {

struct TileChoice {
    int tx, ty, zchunk, graph_steps;
};

struct Tuning {
    // key: (precision, ndim, size class = ceil(log2 n)); the WENO order and
    // the boundary condition share an entry (the last autotune wins)
    std::map<std::tuple<int, int, int>, TileChoice> table;

    static int size_class(int n)
    {
        int c = 0;
        while ((1 << c) < n) ++c;
        return c;
    }

    // The entry that applies to a run whose largest grid has n cells per side,
    // or null.
    const TileChoice* entry(int precision, int ndim, int n) const
    {
        auto it = table.find(std::make_tuple(precision, ndim, size_class(n)));
        return it != table.end() ? &it->second : nullptr;
    }

    // The tiling of a run of count samples: the entry that was set, else the
    // default.  most_tiles: the tiles that the caller has room for (the default
    // keeps to it where a tiling of no more tiles than general()'s does).
    TileChoice choose(int precision, int ndim, const int* sizes, int count, int64_t most_tiles = INT64_MAX) const
    {
        const TileChoice* set = entry(precision, ndim, *std::max_element(sizes, sizes + count));
        return set ? *set : fastest(precision, ndim, sizes, count, most_tiles);
    }

    // The default: the tiling with the least estimated time of a stage launch
    // over all the samples of a run.
    //
    // A workgroup takes `z` planes of its tile one after the other, plus `ends`
    // planes' work at the chunk's two ends (its latency counts less where a CU
    // holds few workgroups), and a CU holding b of them takes slope * b + base
    // times as long as one alone, since they hide each other's latency.  So
    // where the tiles are few, shorter chunks on more CUs finish first; where
    // they fill the GPU many times over, long chunks save the ends; in
    // between, the last round's fill decides.
    // Measured for 4 steps of one sample with WENO5 (us), 16 planes a chunk
    // against the choice here: float 48^3 1748 -> 370, 64^3 1744 -> 504, 96^3
    // 1766 -> 1019, 150^3 3939 -> 3079, 200^3 7168 -> 6626, 256^3 the same;
    // double 48^3 1988 -> 547, 64^3 2010 -> 779, 96^3 2033 -> 1646, 150^3 7144
    // -> 6300, 200^3 the same.
    // A sample's state and step sizes are the same bit for bit under every
    // tiling, and so are its sensors' sums to all but vanishing odds (Sum2), so
    // that the choice can follow a batch's total and the members that are left.
    static TileChoice fastest(int precision, int ndim, const int* sizes, int count, int64_t most_tiles)
    {
        const int maxn = *std::max_element(sizes, sizes + count);
        TileChoice t = general(precision, ndim, maxn);
        if (maxn > kMostCells) return t;            // no solve takes it
        const bool dbl = precision == 1;
        const auto tiles = [&](int tx, int ty, int z) {
            int64_t k = 0;
            for (int i = 0; i < count; ++i)
                k += (int64_t)((sizes[i] + tx - 1) / tx) * (ndim < 2 ? 1 : (sizes[i] + ty - 1) / ty) *
                     (ndim < 3 ? 1 : (sizes[i] + z - 1) / z);
            return k;
        };
        if (ndim == 1) {
            // 4 steps with 64 cells a tile against 256 (us): 64 cells 188
            // against 197, 256 194 and 204, 4000 189 and 196
            if (tiles(64, 1, 1) <= most_tiles) t.tx = 64;
            return t;
        }
        if (ndim == 2) {
            // double: 16 x 8 tiles, whose workgroups take both axes at once, up
            // to one a CU, and up to two where the 16 x 14 ones, which redo less
            // of their halos, would be more than one too (4 steps, us, 16 x 8
            // against 16 x 14: 100^2 233 and 244, 176^2 235 and 251; 192^2 261
            // and 252, 224^2 263 and 252; 240^2 266 and 293, 256^2 266 and 294;
            // 272^2 317 and 295).  float: 16 x 16 where that saves a second
            // tile a CU (256^2 218 against 236; 160^2 216 and 211, 320^2 252
            // and 237).
            if (dbl) {
                const int64_t t8 = tiles(16, 8, 1);
                t.ty = t8 <= most_tiles && (t8 <= kCUs || (t8 <= 2 * kCUs && tiles(16, 14, 1) > kCUs)) ? 8 : 14;
            }
            else t.ty = tiles(16, 16, 1) <= kCUs && tiles(16, 14, 1) > kCUs ? 16 : 14;
            return t;
        }
        const double slope = dbl ? 0.81 : 0.48, base = dbl ? 0.0 : 0.35, least = dbl ? 1.1 : 1.0;
        double best = INFINITY;
        for (int ty : { 14, 16 })
            for (int z : { 32, 24, 16, 12, 8, 6, 4, 3, 2, 1 }) {
                const int64_t n_tiles = tiles(16, ty, z);
                if (n_tiles > std::min(kMaxTiles, most_tiles)) continue;
                // a plane of a 16 x 16 tile against one of 16 x 14: more cells,
                // but (in double above all) less of the GPU's latency hidden
                const double plane = ty == 14 ? 1.0 : dbl ? 1.35 : 1.17;
                const double b = (double)((n_tiles + kCUs - 1) / kCUs);
                const double ends = 0.1 + (dbl ? 0.5 : 0.7) * (1.0 - 1.0 / b);
                const double cost = plane * (z + ends) * std::max(slope * b + base, least);
                if (cost < best) {
                    best = cost;
                    t.ty = ty;
                    t.zchunk = z;
                }
            }
        return t;
    }

    // The tiling by the largest grid alone: of runs where every other would
    // have more than kMaxTiles, or more than there is room for.
    static TileChoice general(int precision, int ndim, int maxn)
    {
        TileChoice t;
        if (ndim == 3) {
            t.tx = 16;
            t.ty = precision == 1 || maxn >= 512 ? 14 : 16;
            t.zchunk = maxn >= 512 ? 32 : 16;
        } else if (ndim == 2) {
            t.tx = 16;
            t.ty = 14;
            t.zchunk = 1;
        } else {
            t.tx = 256;
            t.ty = 1;
            t.zchunk = 1;
        }
        t.graph_steps = maxn >= 256 ? 4 : 16;
        return t;
    }

    static constexpr int kCUs = 256;            // of the GPU
    static constexpr int kMostCells = 4096;     // per side of a grid
    // of the tilings among which the default is chosen (2.3 MB of partials)
    static constexpr int64_t kMaxTiles = 32768;

    void set(int precision, int ndim, int n, const TileChoice& t)
    {
        table[std::make_tuple(precision, ndim, size_class(n))] = t;
    }

    void erase(int precision, int ndim, int n) { table.erase(std::make_tuple(precision, ndim, size_class(n))); }
};

}  // namespace ofm
