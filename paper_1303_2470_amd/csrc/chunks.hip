// Tables of the gathered-chunk step kernel (variant 8), built on the device:
// the tile-ordered compact numbering of the fluid nodes, the chunks of
// consecutive compact nodes, each chunk's halo as a list of 4-node quads, and
// every node's 18 arrival slots. A geometry's tables depend on its node
// classes only.
//
// On the host (one core, a sort per chunk) they took 40 ms for a 64^3 medium
// and were most of a short run; here a chunk is one block, whose halo is
// deduplicated in an LDS hash table and sorted there.
#include "lbmp_internal.hpp"
#include "plan.hpp"

namespace lbmp {
namespace {

constexpr int TT = 256;          // threads per ordering tile
constexpr int CT = 512;          // threads per chunk
constexpr int HTAB = 4096;       // hash slots of a chunk's halo
constexpr int HMAX = 2000;       // halo nodes beyond which no chunk fits: 4 * (511 - 64 / 4) = 1,980 at its shortest
constexpr int HSORT = 2048;

// Fluid and interfacial nodes of every ordering tile.
__global__ void __launch_bounds__(TT) k_tile_count(const int8_t* __restrict__ cls, Order o, uint32_t* __restrict__ cf,
                                                   uint32_t* __restrict__ ci) {
    __shared__ uint32_t sf, si;
    if (threadIdx.x == 0) sf = si = 0;
    __syncthreads();
    const int vol = o.tx * o.ty * o.tz;
    for (int p0 = 0; p0 < vol; p0 += TT) {
        const int p = p0 + threadIdx.x;
        const int64_t n = p < vol ? tile_node(o, blockIdx.x, p) : -1;
        const int c = n >= 0 ? cls[n] : 0;
        const uint64_t bf = __ballot(c != 0), bi = __ballot(c == 2);
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&sf, (uint32_t)__popcll(bf));
            atomicAdd(&si, (uint32_t)__popcll(bi));
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        cf[blockIdx.x] = sf;
        ci[blockIdx.x] = si;
    }
}

// Compact index of every fluid node (lattice order within a tile, tiles from
// the scanned counts), and of every interfacial node among the interfacial ones.
__global__ void __launch_bounds__(TT) k_tile_rank(const int8_t* __restrict__ cls, const int32_t* __restrict__ slot,
                                                  Order o, const uint32_t* __restrict__ of,
                                                  const uint32_t* __restrict__ oi, int32_t* __restrict__ gidx,
                                                  int32_t* __restrict__ gnode, int32_t* __restrict__ gaslot,
                                                  int32_t* __restrict__ aperm) {
    __shared__ uint32_t wf[TT / 64], wi[TT / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint64_t below = (1ull << lane) - 1;
    uint32_t f0 = of[blockIdx.x], i0 = oi[blockIdx.x];
    const int vol = o.tx * o.ty * o.tz;
    for (int p0 = 0; p0 < vol; p0 += TT) {
        const int p = p0 + threadIdx.x;
        const int64_t n = p < vol ? tile_node(o, blockIdx.x, p) : -1;
        const int c = n >= 0 ? cls[n] : 0;
        const uint64_t bf = __ballot(c != 0), bi = __ballot(c == 2);
        if (lane == 0) {
            wf[wv] = (uint32_t)__popcll(bf);
            wi[wv] = (uint32_t)__popcll(bi);
        }
        __syncthreads();
        uint32_t f = f0 + (uint32_t)__popcll(bf & below), i = i0 + (uint32_t)__popcll(bi & below);
        for (int w = 0; w < TT / 64; ++w) {
            if (w < wv) {
                f += wf[w];
                i += wi[w];
            }
            f0 += wf[w];
            i0 += wi[w];
        }
        if (n >= 0) gidx[n] = c ? (int32_t)f : -1;
        if (c) {
            gnode[f] = (int32_t)n;
            gaslot[f] = c == 2 ? (int32_t)i : -1;
            if (c == 2) aperm[slot[n]] = (int32_t)i;
        }
        __syncthreads();
    }
}

struct Halo {  // a chunk's halo in LDS
    int tab[HTAB];
    int hs[HSORT];        // its nodes (compact indices), ascending
    uint16_t qi[HSORT];   // the quad of each
    int cnt, cnt2;
    int wsum[CT / 64];
};

// The arrivals r - c_k of compact node i: compact index, -1 when solid.
struct Pull {
    int x, y, z;
    __device__ __forceinline__ Pull(const Order& o, int n) {
        x = n % o.nx;
        y = (n / o.nx) % o.ny;
        z = n / (o.nx * o.ny);
    }
    __device__ __forceinline__ int32_t at(const Order& o, const int32_t* __restrict__ gidx, int k) const {
        const int64_t m = (int64_t)wrapi(x - lcx(k), o.nx) +
                          (int64_t)o.nx * (wrapi(y - lcy(k), o.ny) + (int64_t)o.ny * wrapi(z - lcz(k), o.nz));
        return gidx[m];
    }
};

// Halo of the chunk base .. base + C - 1 (C at most CT): its nodes sorted into
// h.hs, covered by quads of 4 consecutive compact nodes, each started at the
// lowest node the quads before leave out (a node 4 or more past its
// predecessor always starts one, so the runs between such nodes are
// independent). Returns the quads, -1 when there are more than HMAX nodes;
// nh receives the nodes.
__device__ int chunk_halo(Halo& h, const Order& o, const int32_t* __restrict__ gnode,
                          const int32_t* __restrict__ gidx, int base, int C, int& nh) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    __syncthreads();
    for (int e = tid; e < HTAB; e += CT) h.tab[e] = -1;
    if (tid == 0) h.cnt = h.cnt2 = 0;
    __syncthreads();
    if (tid < C) {
        const Pull p(o, gnode[base + tid]);
        for (int k = 0; k < NL; ++k) {
            const int32_t j = p.at(o, gidx, k);
            if (j < 0 || (j >= base && j < base + C)) continue;
            // each thread looks at the count before it adds a node, so at most
            // HMAX + CT nodes ever enter and the table always has free slots
            if (*(volatile int*)&h.cnt > HMAX) break;
            uint32_t at = ((uint32_t)j * 2654435761u) >> 20;
            for (int probe = 0; probe < HTAB; ++probe, at = (at + 1) & (HTAB - 1)) {
                const int old = atomicCAS(&h.tab[at], -1, j);
                if (old == -1) atomicAdd(&h.cnt, 1);
                if (old == -1 || old == j) break;
            }
        }
    }
    __syncthreads();
    nh = h.cnt;
    if (nh > HMAX) return -1;
    int P = 1;
    while (P < nh) P *= 2;
    for (int e = tid; e < HTAB; e += CT) {
        const int v = h.tab[e];
        if (v >= 0) h.hs[atomicAdd(&h.cnt2, 1)] = v;
    }
    for (int e = nh + tid; e < P; e += CT) h.hs[e] = INT32_MAX;
    for (int e = tid; e < HSORT; e += CT) h.qi[e] = 0;
    __syncthreads();
    for (int k = 2; k <= P; k *= 2)
        for (int j = k / 2; j > 0; j /= 2) {
            for (int t = tid; t < P / 2; t += CT) {
                const int a = 2 * t - (t & (j - 1)), b = a + j;
                const int va = h.hs[a], vb = h.hs[b];
                if ((va > vb) == ((a & k) == 0)) {
                    h.hs[a] = vb;
                    h.hs[b] = va;
                }
            }
            __syncthreads();
        }
    for (int e = tid; e < nh; e += CT)
        if (e == 0 || h.hs[e] - h.hs[e - 1] >= 4) {
            int cur = h.hs[e];
            h.qi[e] = 1;
            for (int i = e + 1; i < nh && h.hs[i] - h.hs[i - 1] < 4; ++i)
                if (h.hs[i] >= cur + 4) {
                    cur = h.hs[i];
                    h.qi[i] = 1;
                }
        }
    __syncthreads();
    // quad of every node: marks up to and including it, less one
    constexpr int PT = HSORT / CT;
    int v[PT], sum = 0;
    for (int i = 0; i < PT; ++i) {
        sum += h.qi[tid * PT + i];
        v[i] = sum;
    }
    int inc = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64);
        if (lane >= off) inc += u;
    }
    if (lane == 63) h.wsum[wv] = inc;
    __syncthreads();
    int before = inc - sum, total = 0;
    for (int w = 0; w < CT / 64; ++w) {
        if (w < wv) before += h.wsum[w];
        total += h.wsum[w];
    }
    for (int i = 0; i < PT; ++i) h.qi[tid * PT + i] = (uint16_t)(before + v[i] - 1);
    __syncthreads();
    return total;
}

// The longest chunk (up to CH nodes, in steps of 64) that may start at compact
// node 64 b: chunk and halo quads leave the last of the CH quads free. 0: none.
__global__ void __launch_bounds__(CT) k_chunk_len(Order o, const int32_t* __restrict__ gnode,
                                                  const int32_t* __restrict__ gidx, int NF, int CH,
                                                  int32_t* __restrict__ len) {
    __shared__ Halo h;
    const int base = (int)blockIdx.x * STEP;
    int C = min(CH, NF - base), nh;
    for (;;) {
        const int H = chunk_halo(h, o, gnode, gidx, base, C, nh);
        const bool fits = H >= 0 && chunk_fits(C, H, CH);
        if (fits || C <= STEP) {
            if (threadIdx.x == 0) len[blockIdx.x] = fits ? C : 0;
            return;
        }
        C = shorter_chunk(C);
    }
}

// Tables of chunk c = list[c] (first node, nodes).
__global__ void __launch_bounds__(CT) k_chunk_build(Order o, const int32_t* __restrict__ gnode,
                                                    const int32_t* __restrict__ gidx, const int2* __restrict__ list,
                                                    int64_t NF, int CH, int4* __restrict__ gch,
                                                    int32_t* __restrict__ ghsrc, uint16_t* __restrict__ gnbr) {
    __shared__ Halo h;
    __shared__ int hq[CT];
    const int base = list[blockIdx.x].x, C = list[blockIdx.x].y, tid = threadIdx.x;
    int nh;
    const int H = chunk_halo(h, o, gnode, gidx, base, C, nh);
    const int64_t hoff = (int64_t)blockIdx.x * CH;
    for (int e = tid; e < nh; e += CT)
        if (e == 0 || h.qi[e] != h.qi[e - 1]) {
            hq[h.qi[e]] = h.hs[e];
            ghsrc[hoff + h.qi[e]] = h.hs[e];
        }
    if (tid == 0) gch[blockIdx.x] = make_int4(base, C, (int)hoff, H);
    __syncthreads();
    const int Cq = (C + 3) / 4;
    const int nz = min(32, 4 * (CH - Cq - H));  // zero slots to choose from: the region's last ones, 4 or more
    const uint32_t zeros = 0xffffffffu << (32 - nz);
    const Pull p(o, gnode[base + min(tid, C - 1)]);
    for (int k = 0; k < NL; ++k) {
        const int32_t j = tid < C ? p.at(o, gidx, k) : -1;
        int sl = -1;
        if (j >= base && j < base + C) sl = j - base;
        else if (j >= 0) {
            int lo = 0, hi = nh - 1;  // j is one of hs
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (h.hs[mid] < j) lo = mid + 1; else hi = mid;
            }
            const int q = h.qi[lo];
            sl = 4 * (Cq + q) + (j - hq[q]);
        }
        // A link from a solid node reads a slot that the copy leaves at zero.
        // The step kernel's arrival reads are bound by bank conflicts, and one
        // zero for all of them met another lane's bank in nearly every read
        // (3.95 cycles a read, counted over this table as 32 lanes on 32 banks;
        // 2 without conflicts): a zero in a bank that no other lane of the
        // half-wave reads serves all of its solid links (3.36). 256^3, 16
        // species: conflicts 3.26e8 -> 2.37e8 cycles, 1,776 -> 1,746 us a step.
        uint32_t used = sl >= 0 ? 1u << (sl & 31) : 0u;
        for (int m = 1; m < 32; m <<= 1) used |= __shfl_xor(used, m, 64);
        const uint32_t free = zeros & ~used;
        if (sl < 0) sl = 4 * CH - 1 - (free ? __clz(free) : 0);
        if (tid < C) gnbr[(int64_t)k * NF + base + tid] = (uint16_t)sl;
    }
}

}  // namespace

lbmp_status build_chunks(const lbmp_flow* f, const int tile[3], int CH, int64_t cap, void* scratch,
                         size_t scratch_bytes, const ChunkTables& T, hipStream_t s, int64_t* nch) {
    *nch = 0;
    const int64_t NF = f->nf;
    const Order o = make_order(f->nx, f->ny, f->nz, tile[0], tile[1], tile[2]);
    const int64_t nt = (int64_t)o.ntx * o.nty * o.ntz, nb = (NF + STEP - 1) / STEP;
    if (CH > CT || CH * cap > (int64_t)INT32_MAX) return LBMP_OK;  // not offered
    Carver c(scratch, scratch_bytes);
    uint32_t* cf = c.take<uint32_t>(nt);
    uint32_t* ci = c.take<uint32_t>(nt);
    int64_t* tot = c.take<int64_t>(2);
    int32_t* len = c.take<int32_t>(nb);
    int2* list = c.take<int2>(cap);
    if (!c.fits()) return LBMP_OK;
    k_tile_count<<<(unsigned)nt, TT, 0, s>>>(f->d.cls, o, cf, ci);
    scan_counts(cf, ci, (int)nt, tot, s);
    k_tile_rank<<<(unsigned)nt, TT, 0, s>>>(f->d.cls, f->d.slot, o, cf, ci, T.gidx, T.gnode, T.gaslot, T.aperm);
    k_chunk_len<<<(unsigned)nb, CT, 0, s>>>(o, T.gnode, T.gidx, (int)NF, CH, len);
    LBMP_HIP(hipGetLastError());
    std::vector<int32_t> lh(nb);
    LBMP_HIP(hipMemcpyAsync(lh.data(), len, nb * 4, hipMemcpyDeviceToHost, s));
    LBMP_HIP(hipStreamSynchronize(s));
    const std::vector<ChunkSpan> ch = chunk_spans(lh.data(), NF, cap);
    if (ch.empty()) return LBMP_OK;  // does not fit: not offered
    static_assert(sizeof(ChunkSpan) == sizeof(int2), "copied as int2");
    LBMP_HIP(hipMemcpyAsync(list, ch.data(), ch.size() * sizeof(int2), hipMemcpyHostToDevice, s));
    k_chunk_build<<<(unsigned)ch.size(), CT, 0, s>>>(o, T.gnode, T.gidx, list, NF, CH, T.gch, T.ghsrc, T.gnbr);
    LBMP_HIP(hipGetLastError());
    LBMP_HIP(hipStreamSynchronize(s));  // ch is read by the copy
    *nch = (int64_t)ch.size();
    return LBMP_OK;
}

}  // namespace lbmp
