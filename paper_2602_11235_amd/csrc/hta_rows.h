// The mapping of query rows to lanes, shared by the row-stationary kernels (and the units of the brief dK/dV pass).
#pragma once
#include "hta_common.h"

namespace hta {

// Query rows as the row-stationary kernels deal them out: the (row, query head) pairs of a kv head's group, packed -- lane rho of
// a tile is row rho / heads, head rho % heads -- so that a tile's last rows fill whole waves whatever the number of heads,
// and a wave's Q, O rows are contiguous in memory.  A group of more heads than a tile has lanes is cut into chunks.
struct RowMap {
    int heads;        // query heads of a chunk
    int n_chunks;     // chunks per kv head
    int rows;         // query rows per tile
    int n_tiles;      // tiles that the longest user needs
    uint32_t magic;   // 2^20 / heads, rounded up: rho / heads for rho < 1024
};
inline RowMap row_map(int tile_lanes, int32_t Hq, int32_t Hkv, int64_t max_rows) {
    const int r = Hq / Hkv;
    RowMap m;
    m.heads = r < tile_lanes ? r : tile_lanes;
    m.n_chunks = (r + m.heads - 1) / m.heads;
    m.rows = tile_lanes / m.heads;
    m.n_tiles = (int)((max_rows + m.rows - 1) / m.rows);
    m.magic = (1u << 20) / (uint32_t)m.heads + 1u;
    return m;
}
// the rows of one tile: row0, head h0 (first of the chunk) and how many of each exist
struct PackedRows {
    struct Row {
        int row, h;
        bool live;
    };
    int row0, h0, n_rows, h_end;  // n_rows: query rows of the user; h_end: first head behind the chunk
    RowMap map;
    __device__ PackedRows(const RowMap& m, int tile, int chunk, int n_rows_, int g, int r) : n_rows(n_rows_), map(m) {
        row0 = tile * m.rows;
        h0 = g * r + chunk * m.heads;
        h_end = min(h0 + m.heads, (g + 1) * r);
    }
    // lanes that do not exist repeat the last row and head that do; their results are never stored
    __device__ __forceinline__ Row at(int rho) const {
        const int q = (int)(((uint32_t)rho * map.magic) >> 20);
        Row x;
        x.row = row0 + q;
        x.h = h0 + rho - q * map.heads;
        x.live = x.row < n_rows && q < map.rows && x.h < h_end;
        x.row = min(x.row, n_rows - 1);
        x.h = min(x.h, h_end - 1);
        return x;
    }
    // does the tile have a row at or behind lane rho?
    __device__ __forceinline__ bool any_from(int rho) const { return rho < min(n_rows - row0, map.rows) * map.heads; }
};

}  // namespace hta
