// Rules that size work before it is launched, free of HIP so that they can be
// compiled and checked without a GPU.
#pragma once

#include <cstdint>
#include <vector>

namespace lbmp {

// ---------------------------------------------------------------- gathered chunks
// Tiles run x fastest, then along y within a band of BAND tile rows, then
// along z, then over the bands: the chunks that an XCD has in flight form a
// box, and more of each other's halo is still in its L2. A step of 16 species
// on 256^3, tiles of 32 x 4 x 4: 1,827 us and 7.98 GB of HBM traffic in plain
// x, y, z order, 1,812 us and 7.68 GB in bands of 4 (2, 3, 6, 8 rows: 1,832,
// 1,815, 1,810, 1,806 us). Tiles of 32 x 8 x 4 have shorter halos, fewer
// copies: 1,776 us, though 8.06 GB.
constexpr int BAND = 4;

struct Order {  // lattice and ordering tiles
    int nx, ny, nz, tx, ty, tz, ntx, nty, ntz;
};

constexpr Order make_order(int nx, int ny, int nz, int tx, int ty, int tz) {
    tx = tx < nx ? tx : nx;
    ty = ty < ny ? ty : ny;
    tz = tz < nz ? tz : nz;
    return {nx, ny, nz, tx, ty, tz, (nx + tx - 1) / tx, (ny + ty - 1) / ty, (nz + tz - 1) / tz};
}

// Lattice index of position p (x fastest) of ordering tile b, -1 outside the lattice.
constexpr int64_t tile_node(const Order& o, int64_t b, int p) {
    const int64_t per = (int64_t)BAND * o.ntz * o.ntx;  // tiles of a whole band
    const int bd = (int)(b / per), left = o.nty - bd * BAND, rows = left < BAND ? left : BAND;
    const int r = (int)((b - bd * per) / o.ntx), bx = (int)((b - bd * per) % o.ntx);
    const int by = bd * BAND + r % rows, bz = r / rows;
    const int lx = p % o.tx, ly = (p / o.tx) % o.ty, lz = p / (o.tx * o.ty);
    const int x = bx * o.tx + lx, y = by * o.ty + ly, z = bz * o.tz + lz;
    return x < o.nx && y < o.ny && z < o.nz ? x + (int64_t)o.nx * (y + (int64_t)o.ny * z) : -1;
}

constexpr int STEP = 64;  // chunk starts are multiples of this, and so is every length but the last chunk's

// The next shorter length to try for a chunk of C > STEP nodes whose halo does
// not fit: the multiple of STEP below C. (C - STEP would leave the remainder of
// the last stretch, NF - base, in the cut length, and with it the next start
// between two measured ones.)
constexpr int shorter_chunk(int C) { return (C - 1) / STEP * STEP; }

// Whether a chunk of C nodes and H halo quads leaves the last of CH quads free.
constexpr bool chunk_fits(int C, int H, int CH) { return (C + 3) / 4 + H <= CH - 1; }

struct ChunkSpan {
    int base, len;
};
// Chunks of NF compact nodes, len[b] the longest that may start at node STEP b
// (0: none fits). Empty when a stretch has no fitting chunk, when more than cap
// are needed, or for lengths that do not lead from multiple to multiple of STEP
// and end at NF: a chunk beyond NF would read and write past its tables.
inline std::vector<ChunkSpan> chunk_spans(const int32_t* len, int64_t NF, int64_t cap) {
    std::vector<ChunkSpan> ch;
    for (int64_t base = 0; base < NF;) {
        const int C = len[base / STEP];
        if (C <= 0 || base % STEP != 0 || base + C > NF || (int64_t)ch.size() >= cap) return {};
        ch.push_back({(int)base, C});
        base += C;
    }
    return ch;
}

}  // namespace lbmp
