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

// ---------------------------------------------------------------- step kernels
constexpr int BLK = 256;             // threads per block (4 waves)
constexpr int TX = 64, TY = BLK / TX;  // reduction tile of variants 1 to 7
constexpr int RCH = 2048;            // tile partials per block of a series reduction

// A launch takes fewer than 2^32 threads in a dimension; more are refused by the
// runtime, and a candidate of the tuner would be timed without its kernel.
constexpr bool launchable(int64_t blocks, int threads) {
    return blocks > 0 && blocks < ((int64_t)1 << 32) / threads;
}

// chunks reserved per geometry: twice the count of full chunks of the
// smaller block (256 nodes)
constexpr int64_t gather_chunk_cap(int64_t nf) { return 2 * (((nf > 1 ? nf : 1) + BLK - 1) / BLK); }

struct PlanGeom {  // what a step's launch depends on
    int nx, ny, nz, S;
    int64_t nf, nch;  // fluid nodes; chunks of variant 8
    int gnh;          // its threads per block / 256
};

// Reduction tiles of a geometry (variant 8: as many as there may be).
constexpr int64_t plan_tiles(const PlanGeom& g, int variant, int K) {
    const int64_t zb = (g.nz + K - 1) / K;  // K = z-planes per tile (z-segment for variant 2)
    const int64_t xt = (g.nx + TX - 1) / TX;
    // variant 8: up to two reduction tiles (halves) per chunk; chunks are cut
    // shorter where their halo would not fit, up to the capacity reserved
    if (variant == 8) return 2 * gather_chunk_cap(g.nf);
    // variant 3: K reduction tiles (TX x TY) per block of TX x (K TY), one z-plane
    // (variant 5: the same with full rows)
    if (variant == 3 || variant == 5) return K * xt * ((g.ny + K * TY - 1) / (K * TY)) * g.nz;
    // variant 4 (6: full rows, 7: lane compaction): K reduction tiles (TX x TY) per block of K planes
    if (variant == 4 || variant == 6 || variant == 7) return K * xt * ((g.ny + TY - 1) / TY) * zb;
    if (variant == 9) return ((int64_t)g.nx * g.ny * g.nz + BLK - 1) / BLK;
    if (variant == 10) return 1;
    if (variant >= 1) return xt * ((g.ny + TY - 1) / TY) * zb;
    return (((int64_t)g.nx * g.ny + BLK - 1) / BLK) * zb;
}

// Reduction tiles a step leaves partials of.
constexpr int64_t plan_partials(const PlanGeom& g, int variant, int K) {
    return variant == 8 ? g.gnh * g.nch : plan_tiles(g, variant, K);
}

// Groups of species (variants 9, 10: of species and nq / K quantities).
constexpr int plan_groups(const PlanGeom& g, int variant, int K, int gsz, int nq) {
    return variant >= 9 ? g.S * (nq / K) : (g.S + gsz - 1) / gsz;
}

// Blocks of a step: one per tile and group; variants 3-7: one per K tiles;
// variant 8: one per chunk.
constexpr int64_t plan_blocks(const PlanGeom& g, int variant, int K, int gsz, int nq) {
    const int64_t tiles = variant == 8 ? g.nch
                          : variant >= 3 && variant < 8 ? plan_tiles(g, variant, K) / K
                                                        : plan_tiles(g, variant, K);
    return tiles * plan_groups(g, variant, K, gsz, nq);
}

constexpr int plan_threads(int variant, int K, int gnh) {
    switch (variant) {
        case 3: return K == 2 ? 2 * BLK : BLK;
        case 4: case 5: case 7: return 2 * BLK;
        case 6: return K == 4 ? 4 * BLK : 2 * BLK;
        case 8: return gnh * BLK;
        case 10: return 4 * BLK;  // at most
        default: return BLK;
    }
}

// Whether the launch of a step over all n geometries, with the blocks that
// record the sums of the step before, is one the runtime takes.
inline bool plan_launchable(const PlanGeom* g, int n, int variant, int K, int gsz, int nq) {
    int64_t blocks = 0, pairs = 0, most = 1;
    for (int i = 0; i < n; ++i) {
        const int64_t parts = plan_partials(g[i], variant, K);
        blocks += plan_blocks(g[i], variant, K, gsz, nq);
        pairs += g[i].S;
        most = parts > most ? parts : most;
    }
    const int64_t nch = (most + RCH - 1) / RCH;
    return launchable(blocks + pairs + (nch > 1 ? pairs * nch : 0), plan_threads(variant, K, g[0].gnh));
}

}  // namespace lbmp
