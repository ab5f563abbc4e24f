// Host model of the gathered chunks' partition (order of the fluid nodes, halo
// of a stretch, its quads) over the library's own rules (plan.hpp):
//   chunk_partition nx ny nz CH cap < mask (one byte per node, 1 = solid)
// prints N_F and the chunks (start, length).
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

using namespace lbmp;

int main(int argc, char** argv) {
    if (argc != 6) return 2;
    const int nx = atoi(argv[1]), ny = atoi(argv[2]), nz = atoi(argv[3]), CH = atoi(argv[4]);
    const int64_t cap = atoll(argv[5]), N = (int64_t)nx * ny * nz;
    std::vector<unsigned char> solid(N);
    if (fread(solid.data(), 1, N, stdin) != (size_t)N) return 3;
    const Order o = make_order(nx, ny, nz, 32, 8, 4);
    std::vector<int32_t> gidx(N, -1), gnode;
    for (int64_t b = 0; b < (int64_t)o.ntx * o.nty * o.ntz; ++b)
        for (int p = 0; p < o.tx * o.ty * o.tz; ++p) {
            const int64_t n = tile_node(o, b, p);
            if (n >= 0 && !solid[n]) {
                gidx[n] = (int32_t)gnode.size();
                gnode.push_back((int32_t)n);
            }
        }
    const int64_t NF = (int64_t)gnode.size();
    std::vector<int32_t> halo;
    auto quads = [&](int64_t base, int C) {  // quads of the halo of base .. base + C - 1
        halo.clear();
        for (int64_t i = base; i < base + C; ++i) {
            const int n = gnode[i], x = n % nx, y = n / nx % ny, z = n / (nx * ny);
            for (int dz = -1; dz <= 1; ++dz)
                for (int dy = -1; dy <= 1; ++dy)
                    for (int dx = -1; dx <= 1; ++dx) {
                        if (dx * dx + dy * dy + dz * dz > 2) continue;
                        const int64_t m = (x + dx + nx) % nx + (int64_t)nx * ((y + dy + ny) % ny + (int64_t)ny * ((z + dz + nz) % nz));
                        const int32_t j = gidx[m];
                        if (j >= 0 && (j < base || j >= base + C)) halo.push_back(j);
                    }
        }
        std::sort(halo.begin(), halo.end());
        int64_t q = 0, next = -1;
        for (const int32_t h : halo)
            if (h >= next) {
                ++q;
                next = h + 4;
            }
        return (int)q;
    };
    std::vector<int32_t> len;
    for (int64_t base = 0; base < NF; base += STEP) {
        int C = (int)std::min<int64_t>(CH, NF - base);
        bool fits = chunk_fits(C, quads(base, C), CH);
        while (!fits && C > STEP) {
            C = shorter_chunk(C);
            fits = chunk_fits(C, quads(base, C), CH);
        }
        len.push_back(fits ? C : 0);
    }
    printf("%lld\n", (long long)NF);
    for (const ChunkSpan& c : chunk_spans(len.data(), NF, cap)) printf("%d %d\n", c.base, c.len);
    return 0;
}
