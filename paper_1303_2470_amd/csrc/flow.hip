// Steady fluid flow by the lattice-Boltzmann equation (Eq. 6 of the paper):
// D3Q19 BGK, Guo forcing, half-way bounce-back, FP64, fused pull-stream +
// collide, one thread per fluid node, populations ping-pong over the
// fluid nodes only (in lattice order, through a lattice -> compact
// index map), so that no lane idles on a solid node and no solid value is
// moved; velocities are compact too until the reported one.
//
// The stored state is the post-collision population. A step gathers the
// post-collision populations of the upstream neighbours (or the reflected
// population of the node itself when the upstream node is solid), forms the
// density and the force-corrected velocity u = (sum f c)/rho + g/2, and
// relaxes towards the equilibrium with the Guo source term.
#include <cstring>
#include <mutex>
#include <type_traits>

#include "lbmp_internal.hpp"

namespace lbmp {

// Populations are stored in tiles of PT nodes, [tile][19][PT]: a block reads
// and writes one stretch of memory instead of 19 (+ 19) that lie N_F values
// apart (256^3 porous medium: 503 -> 467 us a step; tiles of 64 to 4,096 nodes
// within 1 %). PT = 0, [19][N_F], needs no room for a last tile that is not
// full: for the resident kernel, which loads them once per launch, and for a
// scratch that has no such room (600 steps of 349,500 nodes: 17 ms; node by
// node, [N_F][19], 49 ms).
constexpr int TILE = 256;
__host__ __device__ constexpr int64_t tiled(int64_t nf) { return (nf + TILE - 1) / TILE * TILE; }
template <int PT>
__device__ __forceinline__ int64_t pidx(int k, int64_t i, int64_t NF) {
    if constexpr (PT == 0) return k * NF + i;
    else return (i / PT * 19 + k) * PT + i % PT;
}

struct BGKParams {
    double om, pre;  // 1 / tau, 1 - 1 / (2 tau)
    double gx, gy, gz;
};

// c_k . v, the terms with a zero component left out.
template <typename F>
__device__ __forceinline__ double cdot(int k, F x, F y, F z) {
    double s = 0.0;
    bool first = true;
    auto add = [&](int c, double v) {
        if (c == 0) return;
        s = first ? (c > 0 ? v : -v) : (c > 0 ? s + v : s - v);
        first = false;
    };
    add(lcx(k), x);
    add(lcy(k), y);
    add(lcz(k), z);
    return s;
}

// BGK collision with Guo forcing, every sum and product in the order of
//   feq = w rho (1 + 3 cu + 9/2 cu^2 - 3/2 u^2),
//   S = pre w (3 (cF - uF) + 9 cu cF),  f' = f - om (f - feq) + S,
// written out so that terms with a zero component of c cost nothing (IEEE
// rules keep a product with 0) and the opposite links k, k ^ 1, whose cu and
// cF differ in sign only, share what is even: the same bits at less than half
// the FP64 instructions.
__device__ inline void bgk_collide(double f[19], const BGKParams& P, double& rho, double& ux,
                                   double& uy, double& uz) {
    double r = f[0], jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const double v = f[k + 1];
        r += v;
        if (lcx(k)) jx = lcx(k) > 0 ? jx + v : jx - v;
        if (lcy(k)) jy = lcy(k) > 0 ? jy + v : jy - v;
        if (lcz(k)) jz = lcz(k) > 0 ? jz + v : jz - v;
    }
    rho = r;
    ux = jx / r + 0.5 * P.gx;
    uy = jy / r + 0.5 * P.gy;
    uz = jz / r + 0.5 * P.gz;
    const double Fx = r * P.gx, Fy = r * P.gy, Fz = r * P.gz;
    const double uu = ux * ux + uy * uy + uz * uz;
    const double uF = ux * Fx + uy * Fy + uz * Fz;
    const double om = P.om, pre = P.pre;
    const double uu15 = 1.5 * uu;
    // rest population
    {
        double feq = W_REST * r * (1.0 - uu15);
        double S = pre * W_REST * (-3.0 * uF);
        f[0] = f[0] - om * (f[0] - feq) + S;
    }
#pragma unroll
    for (int k = 0; k < NL; k += 2) {
        const double cu = cdot(k, ux, uy, uz), cF = cdot(k, Fx, Fy, Fz);
        const double c3 = 3.0 * cu, q = 4.5 * cu * cu, uf9 = 9.0 * cu * cF;
        const double wr = lw(k) * r, wp = pre * lw(k);
        const double feq0 = wr * (1.0 + c3 + q - uu15), feq1 = wr * (1.0 - c3 + q - uu15);
        const double S0 = wp * (3.0 * (cF - uF) + uf9), S1 = wp * (3.0 * (-cF - uF) + uf9);
        f[k + 1] = f[k + 1] - om * (f[k + 1] - feq0) + S0;
        f[k + 2] = f[k + 2] - om * (f[k + 2] - feq1) + S1;
    }
}

// Start at rest: equilibrium with rho = 1, u = 0, then one collision with the
// force (the same for every node).
template <int PT>
__global__ void k_bgk_init(double* __restrict__ fo, int64_t NF, BGKParams P, double* __restrict__ u0) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NF) return;
    double f[19];
    f[0] = W_REST;
#pragma unroll
    for (int k = 0; k < NL; ++k) f[k + 1] = lw(k);
    double rho, ux, uy, uz;
    bgk_collide(f, P, rho, ux, uy, uz);
    for (int k = 0; k < 19; ++k) fo[pidx<PT>(k, i, NF)] = f[k];
    u0[i] = ux;
    u0[NF + i] = uy;
    u0[2 * NF + i] = uz;
}

// Compact index of the node r - c_k for every link of lattice node n (32-bit
// index arithmetic; the host bounds N), -1 where it is solid.
struct Upstream {
    uint32_t xo[3], yo[3], zo[3];
    __device__ __forceinline__ Upstream(uint32_t n, uint32_t nx, uint32_t ny, uint32_t nz) {
        const uint32_t plane = nx * ny, z = n / plane, r = n - z * plane, y = r / nx, x = r - y * nx;
        xo[0] = x == 0 ? nx - 1 : x - 1;
        xo[1] = x;
        xo[2] = x + 1 == nx ? 0 : x + 1;
        yo[0] = (y == 0 ? ny - 1 : y - 1) * nx;
        yo[1] = y * nx;
        yo[2] = (y + 1 == ny ? 0 : y + 1) * nx;
        zo[0] = (z == 0 ? nz - 1 : z - 1) * plane;
        zo[1] = z * plane;
        zo[2] = (z + 1 == nz ? 0 : z + 1) * plane;
    }
    __device__ __forceinline__ int32_t at(const int32_t* __restrict__ gidx, int k) const {
        return gidx[zo[1 - lcz(k)] + yo[1 - lcy(k)] + xo[1 - lcx(k)]];
    }
};

// Where every population is pulled from, for lattices that take the table:
// pull[k][i] = index of the stored population that becomes k + 1 of node i (the
// upstream node's, or the node's own reflected one).
__global__ void k_bgk_table(const int32_t* __restrict__ gnode, const int32_t* __restrict__ gidx, int64_t NF, int nx,
                            int ny, int nz, int32_t* __restrict__ pull) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NF) return;
    const Upstream up((uint32_t)gnode[i], nx, ny, nz);
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int32_t j = up.at(gidx, k);
        pull[k * NF + i] = (int32_t)(j < 0 ? pidx<TILE>((k ^ 1) + 1, i, NF) : pidx<TILE>(k + 1, j, NF));
    }
}

// One step for fluid node i (lattice index gnode[i]): pull, collide, store.
// TAB: through the table; otherwise through the compact map gidx (-1 on solid
// nodes: the node's own reflected population instead). Blocks are remapped so
// that each XCD takes a contiguous range of nodes and the rows and planes that
// neighbouring blocks look up in gidx are found in its own L2. Large lattices
// are bound by HBM: 467 us for 6.71 M nodes, 304 B each, is 4.4 TB/s, where a
// copy reaches 4.9-5.2 (540 us before the tiles, the remap and the shorter
// collision). Small ones, held by the last-level
// cache, are bound by its bandwidth and by the chain of dependent loads.
template <bool TAB, int PT>
__global__ void __launch_bounds__(256) k_bgk_step(const int32_t* __restrict__ gnode, const int32_t* __restrict__ gidx,
                                                  const int32_t* __restrict__ pull, const double* __restrict__ fi,
                                                  double* __restrict__ fo, int64_t NF, int nx, int ny, int nz,
                                                  BGKParams P, double* __restrict__ uout) {
    const unsigned nb = gridDim.x, per = nb / 8, rem = nb % 8, xcd = blockIdx.x % 8;
    const int64_t blk = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + blockIdx.x / 8;
    const int64_t i = blk * blockDim.x + threadIdx.x;
    if (i >= NF) return;
    double f[19];
    f[0] = fi[pidx<PT>(0, i, NF)];
    if constexpr (TAB) {
        int32_t at[NL];
#pragma unroll
        for (int k = 0; k < NL; ++k) at[k] = pull[k * NF + i];
#pragma unroll
        for (int k = 0; k < NL; ++k) f[k + 1] = fi[at[k]];
    } else {
        const Upstream up((uint32_t)gnode[i], nx, ny, nz);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int32_t j = up.at(gidx, k);
            f[k + 1] = fi[j < 0 ? pidx<PT>((k ^ 1) + 1, i, NF) : pidx<PT>(k + 1, (uint32_t)j, NF)];
        }
    }
    double rho, ux, uy, uz;
    bgk_collide(f, P, rho, ux, uy, uz);
#pragma unroll
    for (int k = 0; k < 19; ++k) fo[pidx<PT>(k, i, NF)] = f[k];
    if (uout) {
        uout[i] = ux;
        uout[NF + i] = uy;
        uout[2 * NF + i] = uz;
    }
}

// Maximum of d >= 0 and x >= 0; infinite once x is not finite (fmax drops a
// NaN, and a flow that is NaN everywhere would have a residual of zero).
__device__ __forceinline__ double fmax_finite(double d, double x) { return x < INFINITY ? fmax(d, x) : INFINITY; }

// Lattices of at most BRES_NODES fluid nodes: the whole solve in one block,
// populations in LDS (152 B a node), one node per thread, until the residual
// falls below tol or nsteps are done. A launch per step cost 5.7 us however
// small the lattice. Arithmetic and its order are those of k_bgk_step and
// k_resid. st: steps done so far, then 1 once converged (2: non-finite).
// F: the stored populations; U: velocities of the last three steps, slot =
// step % 3.
constexpr int BRES_NODES = 1024;
constexpr int BRES_STEPS = 20000;  // per launch

template <int BS>
__global__ void __launch_bounds__(BS) k_bgk_resident(const int32_t* __restrict__ gnode, const int32_t* __restrict__ gidx,
                                                     int NF, int nx, int ny, int nz, BGKParams P, double tol, int ce,
                                                     int nsteps, double* __restrict__ F, double* __restrict__ U0,
                                                     double* __restrict__ U1, double* __restrict__ U2,
                                                     double* __restrict__ res, int64_t* __restrict__ st) {
    __shared__ double pop[19 * BS];
    __shared__ double sd[BS / 64], sm[BS / 64];
    double* const U[3] = {U0, U1, U2};
    const int i = threadIdx.x, lane = i & 63, wv = i >> 6;
    const bool act = i < NF;
    const int64_t step0 = st[0];
    int at[NL];
    {
        const Upstream up(act ? (uint32_t)gnode[i] : 0u, nx, ny, nz);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int32_t j = act ? up.at(gidx, k) : -1;
            at[k] = j < 0 ? ((k ^ 1) + 1) * BS + i : (k + 1) * BS + j;
        }
    }
    // lanes without a node carry the state at rest along
#pragma unroll
    for (int k = 0; k < 19; ++k) pop[k * BS + i] = act ? F[pidx<0>(k, i, NF)] : (k == 0 ? W_REST : lw(k - 1));
    // velocities of the last step (slot step0 % 3) and the one before
    const int s0 = (int)(step0 % 3);
    double ua[3], ub[3], uc[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        ua[d] = act ? U[s0][d * NF + i] : 0.0;
        ub[d] = act && step0 > 0 ? U[(s0 + 2) % 3][d * NF + i] : 0.0;
        uc[d] = 0.0;
    }
    int phase = (int)(step0 % ce), done = 0, verdict = 0;
    bool checked = false;
    double rd = 0.0, rm = 0.0;
    while (done < nsteps && verdict == 0) {
        __syncthreads();
        double f[19];
        f[0] = pop[i];
#pragma unroll
        for (int k = 0; k < NL; ++k) f[k + 1] = pop[at[k]];
        __syncthreads();
        double rho, ux, uy, uz;
        bgk_collide(f, P, rho, ux, uy, uz);
#pragma unroll
        for (int k = 0; k < 19; ++k) pop[k * BS + i] = f[k];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            uc[d] = ub[d];
            ub[d] = ua[d];
        }
        ua[0] = ux;
        ua[1] = uy;
        ua[2] = uz;
        ++done;
        if (++phase == ce) {
            phase = 0;
            if (step0 + done >= 2) {
                double d = 0.0, m = 0.0;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double a = 0.5 * (ua[k] + ub[k]), b = 0.5 * (ub[k] + uc[k]);
                    d = fmax_finite(d, act ? fabs(a - b) : 0.0);
                    m = fmax(m, act ? fabs(a) : 0.0);
                }
                for (int s = 32; s > 0; s >>= 1) {
                    d = fmax(d, __shfl_xor(d, s, 64));
                    m = fmax(m, __shfl_xor(m, s, 64));
                }
                if (lane == 0) {
                    sd[wv] = d;
                    sm[wv] = m;
                }
                __syncthreads();
                rd = sd[0];
                rm = sm[0];
                for (int w = 1; w < BS / 64; ++w) {
                    rd = fmax(rd, sd[w]);
                    rm = fmax(rm, sm[w]);
                }
                const double v = rm > 0.0 ? rd / rm : rd;
                verdict = !isfinite(v) ? 2 : v < tol ? 1 : 0;
                checked = true;
                __syncthreads();
            }
        }
    }
    const int s1 = (int)((step0 + done) % 3);
    if (act) {
#pragma unroll
        for (int k = 0; k < 19; ++k) F[pidx<0>(k, i, NF)] = pop[k * BS + i];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            U[s1][d * NF + i] = ua[d];
            U[(s1 + 2) % 3][d * NF + i] = ub[d];
        }
    }
    if (i == 0) {
        if (checked) {
            res[0] = rd;
            res[1] = rm;
        }
        st[0] = step0 + done;
        st[1] = verdict;
    }
}

// Block maxima of |ubar(t) - ubar(t-1)| (infinite where a component is not
// finite) and |ubar(t)| over all components, ubar(t) = (u(t) + u(t-1))/2, from
// the velocities of the last three steps.
__global__ void __launch_bounds__(256) k_resid(const double* __restrict__ u2, const double* __restrict__ u1,
                                               const double* __restrict__ u0, int64_t n3, double* __restrict__ part) {
    __shared__ double sd[256], sm[256];
    double d = 0.0, m = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n3;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double a = 0.5 * (u0[i] + u1[i]), b = 0.5 * (u1[i] + u2[i]);
        d = fmax_finite(d, fabs(a - b));
        m = fmax(m, fabs(a));
    }
    sd[threadIdx.x] = d;
    sm[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sd[threadIdx.x] = fmax(sd[threadIdx.x], sd[threadIdx.x + s]);
            sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = sd[0];
        part[2 * blockIdx.x + 1] = sm[0];
    }
}

// Maxima over the nb block maxima, in one wave (one thread walking them took
// 54 us of every check).
__global__ void __launch_bounds__(64) k_resid_final(const double* __restrict__ part, int nb, double* __restrict__ out) {
    double d = 0.0, m = 0.0;
    for (int k = threadIdx.x; k < nb; k += 64) {
        d = fmax(d, part[2 * k]);
        m = fmax(m, part[2 * k + 1]);
    }
    for (int s = 32; s > 0; s >>= 1) {
        d = fmax(d, __shfl_xor(d, s, 64));
        m = fmax(m, __shfl_xor(m, s, 64));
    }
    if (threadIdx.x == 0) {
        out[0] = d;
        out[1] = m;
    }
}

// Reported velocity on the lattice: average of the last two steps, zero on solid nodes.
__global__ void k_uavg(const double* __restrict__ u1, const double* __restrict__ u0, const int32_t* __restrict__ gidx,
                       int64_t N, int64_t NF, double* __restrict__ out) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    const int64_t i = gidx[n];
#pragma unroll
    for (int d = 0; d < 3; ++d) out[d * N + n] = i < 0 ? 0.0 : 0.5 * (u0[d * NF + i] + u1[d * NF + i]);
}

__global__ void k_zero_solid_u(const uint8_t* __restrict__ solid, double* __restrict__ u, int64_t N) {
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    if (solid[n]) u[n] = u[N + n] = u[2 * N + n] = 0.0;
}

constexpr int RES_BLOCKS = 512;
// The pull table replaces two dependent loads and the index arithmetic by one
// streamed load of 72 B a node: worth it while the whole solve stays in cache
// and latency counts, not beyond. us a step with and without it, by fluid
// nodes: 33,792 5.5 and 7.8, 103,680 8.2 and 11.0, 192,512 12.7 and 14.3,
// 225,280 14.3 and 15.4, 252,599 (porous) 16.1 and 15.9, 357,696 21.0 and 19.3.
constexpr int64_t TABLE_NODES = 3 << 16;

// what a solve needs; room for full tiles and the pull table on top of it
static size_t scratch_bytes_for(int64_t N) {
    return 2 * align_up(19 * 8 * (size_t)N) + 3 * align_up(24 * (size_t)N) +
           align_up(2 * 8 * RES_BLOCKS) + align_up(16) + 2 * align_up(4 * (size_t)N);
}
static size_t tile_bytes_for(int64_t NF) {
    return 2 * (align_up(19 * 8 * (size_t)tiled(NF)) - align_up(19 * 8 * (size_t)NF));
}
static size_t table_bytes_for(int64_t NF) { return align_up(4 * NL * (size_t)NF); }

}  // namespace lbmp

using namespace lbmp;

extern "C" lbmp_status lb_flow_workspace_bytes(const lbmp_geometry* g, size_t* persistent,
                                               size_t* scratch_out) {
    if (!g || g->nx <= 0 || g->ny <= 0 || g->nz <= 0)
        return fail(LBMP_EINVAL, "invalid geometry");
    int64_t N = (int64_t)g->nx * g->ny * g->nz;
    if (persistent) *persistent = align_up(sizeof(lbmp_flow)) + geometry_bytes(N);
    if (scratch_out) *scratch_out = scratch_bytes_for(N) + tile_bytes_for(N) + (N <= TABLE_NODES ? table_bytes_for(N) : 0);
    return LBMP_OK;
}

static lbmp_status make_flow(const lbmp_geometry* g, void* dev_ws, size_t ws_bytes, hipStream_t s,
                             lbmp_flow** out) {
    lbmp_status st = validate_geometry(g);
    if (st != LBMP_OK) return st;
    if (!dev_ws) return fail(LBMP_EINVAL, "workspace is NULL");
    int64_t N = (int64_t)g->nx * g->ny * g->nz;
    Carver c(dev_ws, ws_bytes);
    c.take<char>(sizeof(lbmp_flow));  // reserved, keeps layouts aligned with the query
    auto* f = new lbmp_flow();
    f->magic = FLOW_MAGIC;
    f->nx = g->nx;
    f->ny = g->ny;
    f->nz = g->nz;
    f->nbhd = g->iface_nbhd == 6 ? 6 : 18;
    f->N = N;
    st = build_geometry(g, c, f->d, s, &f->nf, &f->ni);
    if (st != LBMP_OK) {
        delete f;
        return st;
    }
    f->converged = 1;
    f->steps = 0;
    f->residual = 0.0;
    *out = f;
    return LBMP_OK;
}

// The solve of lb_flow_solve and lb_flow_solve_static: populations, velocity
// history and residual partials in dev_scratch (scratch_bytes long); nothing
// in dev_scratch needs to start at zero.
static lbmp_status flow_solve(const lbmp_geometry* g, double tau, const double force[3], double tol,
                              int64_t max_steps, int check_every, void* dev_ws, size_t ws_bytes,
                              void* dev_scratch, size_t scratch_bytes, void* hip_stream, lbmp_flow** out,
                              int64_t* steps_done, double* residual) {
    if (!out) return fail(LBMP_EINVAL, "out is NULL");
    *out = nullptr;
    if (!(tau > 0.5) || !std::isfinite(tau)) return fail(LBMP_EINVAL, "tau must exceed 1/2");
    if (!force || !std::isfinite(force[0]) || !std::isfinite(force[1]) || !std::isfinite(force[2]))
        return fail(LBMP_EINVAL, "force must be finite");
    if (max_steps < 1) return fail(LBMP_EINVAL, "max_steps must be >= 1");
    if (!(tol >= 0.0)) return fail(LBMP_EINVAL, "tol must be >= 0");
    if (check_every < 0) return fail(LBMP_EINVAL, "check_every must be >= 0");
    int ce = check_every == 0 ? 100 : check_every;
    lbmp_status st = validate_geometry(g);
    if (st != LBMP_OK) return st;
    size_t need_p = 0;
    st = lb_flow_workspace_bytes(g, &need_p, nullptr);
    if (st != LBMP_OK) return st;
    const size_t need_s = scratch_bytes_for((int64_t)g->nx * g->ny * g->nz);
    if (ws_bytes < need_p || scratch_bytes < need_s || !dev_scratch)
        return fail(LBMP_ENOMEM, "workspace %zu/%zu bytes, need %zu/%zu", ws_bytes, scratch_bytes,
                    need_p, need_s);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    lbmp_flow* f = nullptr;
    st = make_flow(g, dev_ws, ws_bytes, s, &f);
    if (st != LBMP_OK) return st;
    const int64_t N = f->N, NF = f->nf, n3 = 3 * NF;
    Carver c(dev_scratch, scratch_bytes);
    const bool resident = NF <= BRES_NODES;
    // (U, part, res, gidx and gnode take what scratch_bytes_for counts, for NF
    // fluid nodes of N)
    const bool tiles = !resident && scratch_bytes_for(NF) + 2 * (align_up(4 * (size_t)N) - align_up(4 * (size_t)NF)) +
                                        tile_bytes_for(NF) <= scratch_bytes;
    double* fa = c.take<double>(19 * (tiles ? tiled(NF) : NF));
    double* fb = c.take<double>(19 * (tiles ? tiled(NF) : NF));
    // velocities of the last three steps, slot = step % 3
    double* U[3] = {c.take<double>(n3), c.take<double>(n3), c.take<double>(n3)};
    double* part = c.take<double>(2 * RES_BLOCKS);
    double* res = c.take<double>(4);  // the last two for k_bgk_resident's counters
    int32_t* gidx = c.take<int32_t>(N);
    int32_t* gnode = c.take<int32_t>(N);
    rank_fluid(f, gidx, gnode, s);
    const unsigned nbf = (unsigned)((NF + 255) / 256);
    const bool tab = tiles && NF <= TABLE_NODES && c.off + table_bytes_for(NF) <= scratch_bytes;
    int32_t* const pull = tab ? c.take<int32_t>(NL * NF) : nullptr;
    if (tab) k_bgk_table<<<nbf, 256, 0, s>>>(gnode, gidx, NF, f->nx, f->ny, f->nz, pull);
    BGKParams P{1.0 / tau, 1.0 - 0.5 / tau, force[0], force[1], force[2]};
    if (tiles) k_bgk_init<TILE><<<nbf, 256, 0, s>>>(fa, NF, P, U[0]);
    else k_bgk_init<0><<<nbf, 256, 0, s>>>(fa, NF, P, U[0]);
    // before step 2 the history holds the start only
    LBMP_HIP(hipGetLastError());
    double resv = INFINITY;
    int64_t step = 0;
    int conv = 0;
    if (resident) {
        int64_t* const st_dev = reinterpret_cast<int64_t*>(res + 2);
        LBMP_HIP(hipMemsetAsync(res, 0, 32, s));
        int verdict = 0;
        while (step < max_steps && verdict == 0) {
            const int n = (int)std::min<int64_t>(BRES_STEPS, max_steps - step);
            auto go = [&](auto bs) {
                constexpr int BS = decltype(bs)::value;
                k_bgk_resident<BS><<<1, BS, 0, s>>>(gnode, gidx, (int)NF, f->nx, f->ny, f->nz, P, tol, ce, n, fa, U[0],
                                                    U[1], U[2], res, st_dev);
            };
            if (NF <= 64) go(std::integral_constant<int, 64>());
            else if (NF <= 128) go(std::integral_constant<int, 128>());
            else if (NF <= 256) go(std::integral_constant<int, 256>());
            else if (NF <= 512) go(std::integral_constant<int, 512>());
            else go(std::integral_constant<int, 1024>());
            LBMP_HIP(hipGetLastError());
            double h[4];
            LBMP_HIP(hipMemcpyAsync(h, res, sizeof h, hipMemcpyDeviceToHost, s));
            LBMP_HIP(hipStreamSynchronize(s));
            int64_t c2[2];
            memcpy(c2, h + 2, sizeof c2);
            step = c2[0];
            verdict = (int)c2[1];
            if (step / ce * ce >= 2) resv = h[1] > 0.0 ? h[0] / h[1] : h[0];  // a check was made
        }
        conv = verdict == 1;
        if (verdict == 2) {
            delete f;
            return fail(LBMP_ENUMERIC, "flow solve produced a non-finite velocity at step %lld", (long long)step);
        }
    }
    while (!resident && step < max_steps) {
        const int64_t sn = step + 1;
        const bool check = sn >= 2 && (sn % ce) == 0;
        // u is needed at a check step and the two steps before it, and at the
        // last two steps (the reported velocity)
        const bool need = check || ((sn + 1) % ce) == 0 || ((sn + 2) % ce) == 0 || sn + 1 >= max_steps;
        double* uo = need ? U[sn % 3] : nullptr;
        auto go = [&](auto tabc, auto ptc) {
            k_bgk_step<decltype(tabc)::value, decltype(ptc)::value>
                <<<nbf, 256, 0, s>>>(gnode, gidx, pull, fa, fb, NF, f->nx, f->ny, f->nz, P, uo);
        };
        if (tab) go(std::true_type(), std::integral_constant<int, TILE>());
        else if (tiles) go(std::false_type(), std::integral_constant<int, TILE>());
        else go(std::false_type(), std::integral_constant<int, 0>());
        std::swap(fa, fb);
        step = sn;
        if (check) {
            k_resid<<<RES_BLOCKS, 256, 0, s>>>(U[(sn - 2) % 3], U[(sn - 1) % 3], U[sn % 3], n3, part);
            k_resid_final<<<1, 64, 0, s>>>(part, RES_BLOCKS, res);
            double h[2];
            LBMP_HIP(hipMemcpyAsync(h, res, sizeof h, hipMemcpyDeviceToHost, s));
            LBMP_HIP(hipStreamSynchronize(s));
            resv = h[1] > 0.0 ? h[0] / h[1] : h[0];
            if (!std::isfinite(resv)) {
                delete f;
                return fail(LBMP_ENUMERIC, "flow solve produced a non-finite velocity at step %lld",
                            (long long)sn);
            }
            if (resv < tol) {
                conv = 1;
                break;
            }
        }
    }
    LBMP_HIP(hipGetLastError());
    {
        // step >= 1: u(step) and u(step-1) were both written (u(0) by the init)
        k_uavg<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(U[(step - 1) % 3], U[step % 3], gidx, N, NF, f->d.u);
        LBMP_HIP(hipGetLastError());
    }
    LBMP_HIP(hipStreamSynchronize(s));
    f->converged = conv;
    f->steps = step;
    f->residual = resv;
    if (steps_done) *steps_done = step;
    if (residual) *residual = resv;
    *out = f;
    if (!conv) return fail(LBMP_ENOTCONV, "flow not converged after %lld steps (residual %.3e)",
                           (long long)step, resv);
    return LBMP_OK;
}

extern "C" lbmp_status lb_flow_solve(const lbmp_geometry* g, double tau, const double force[3],
                                     double tol, int64_t max_steps, int check_every, void* dev_ws,
                                     size_t ws_bytes, void* dev_scratch, size_t scratch_bytes,
                                     void* hip_stream, lbmp_flow** out, int64_t* steps_done,
                                     double* residual) {
    return flow_solve(g, tau, force, tol, max_steps, check_every, dev_ws, ws_bytes, dev_scratch, scratch_bytes,
                      hip_stream, out, steps_done, residual);
}

// ---------------------------------------------------------------- no-allocation solve
// lb_flow_solve_static takes its scratch from a file-scope device array
// instead of a caller workspace, for callers that cannot allocate device
// memory. Each GPU holds its own copy of the array (at its own address) until
// the process ends; the host-side name is not a device address, so the
// address is taken once per device with hipGetSymbolAddress and used from
// then on.
namespace lbmp {
static __device__ __align__(256) unsigned char scratch[LBMP_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[MAX_DEVICES];  // per device, null until first use there

static lbmp_status static_scratch(void** ptr) {
    int dev = -1;
    LBMP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(LBMP_EDEVICE, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(LBMP_EDEVICE, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev,
                        hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return LBMP_OK;
}
}  // namespace lbmp

extern "C" lbmp_status lb_flow_solve_static(const lbmp_geometry* g, double tau, const double force[3],
                                            double tol, int64_t max_steps, int check_every, void* dev_ws,
                                            size_t ws_bytes, void* hip_stream, lbmp_flow** out,
                                            int64_t* steps_done, double* residual) {
    if (!out) return fail(LBMP_EINVAL, "out is NULL");
    *out = nullptr;
    lbmp_status st = validate_geometry(g);
    if (st != LBMP_OK) return st;
    const int64_t N = (int64_t)g->nx * g->ny * g->nz;
    const size_t need = scratch_bytes_for(N);
    if (need > (size_t)LBMP_STATIC_SCRATCH_BYTES)
        return fail(LBMP_ENOMEM, "lattice of %lld nodes needs %zu scratch bytes; the static scratch holds %zu "
                    "(at most %lld nodes)", (long long)N, need, (size_t)LBMP_STATIC_SCRATCH_BYTES,
                    (long long)lb_flow_static_max_nodes());
    void* p = nullptr;
    st = static_scratch(&p);
    if (st != LBMP_OK) return st;
    return flow_solve(g, tau, force, tol, max_steps, check_every, dev_ws, ws_bytes, p,
                      (size_t)LBMP_STATIC_SCRATCH_BYTES, hip_stream, out, steps_done, residual);
}

extern "C" int64_t lb_flow_static_max_nodes(void) {
    // scratch_bytes_for is 384 bytes per node plus alignment and the residual
    // partials; the largest N that fits
    int64_t lo = 0, hi = (int64_t)LBMP_STATIC_SCRATCH_BYTES / 384 + 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (scratch_bytes_for(mid) <= (size_t)LBMP_STATIC_SCRATCH_BYTES) lo = mid; else hi = mid - 1;
    }
    return lo;
}

extern "C" lbmp_status lb_flow_from_velocity(const lbmp_geometry* g, const double* u_host,
                                             void* dev_ws, size_t ws_bytes, void* hip_stream,
                                             lbmp_flow** out) {
    if (!out) return fail(LBMP_EINVAL, "out is NULL");
    *out = nullptr;
    if (!u_host) return fail(LBMP_EINVAL, "velocity is NULL");
    lbmp_status st = validate_geometry(g);
    if (st != LBMP_OK) return st;
    size_t need_p = 0;
    st = lb_flow_workspace_bytes(g, &need_p, nullptr);
    if (st != LBMP_OK) return st;
    if (ws_bytes < need_p) return fail(LBMP_ENOMEM, "workspace %zu bytes, need %zu", ws_bytes, need_p);
    int64_t N = (int64_t)g->nx * g->ny * g->nz;
    for (int d = 0; d < 3; ++d)
        for (int64_t i = 0; i < N; ++i)
            if (!std::isfinite(u_host[d * N + i]) && !g->solid[i])
                return fail(LBMP_EINVAL, "velocity is not finite at a fluid node");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    lbmp_flow* f = nullptr;
    st = make_flow(g, dev_ws, ws_bytes, s, &f);
    if (st != LBMP_OK) return st;
    LBMP_HIP(hipMemcpyAsync(f->d.u, u_host, 24 * (size_t)N, hipMemcpyHostToDevice, s));
    k_zero_solid_u<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(f->d.solid, f->d.u, N);
    LBMP_HIP(hipGetLastError());
    LBMP_HIP(hipStreamSynchronize(s));
    *out = f;
    return LBMP_OK;
}

extern "C" lbmp_status lb_flow_velocity(const lbmp_flow* f, double* u_host) {
    if (!f || f->magic != FLOW_MAGIC) return fail(LBMP_ESTATE, "invalid flow handle");
    if (!u_host) return fail(LBMP_EINVAL, "output is NULL");
    LBMP_HIP(hipMemcpy(u_host, f->d.u, 24 * (size_t)f->N, hipMemcpyDeviceToHost));
    return LBMP_OK;
}

extern "C" lbmp_status lb_flow_classes(const lbmp_flow* f, int8_t* cls_host, int64_t* n_fluid,
                                       int64_t* n_iface) {
    if (!f || f->magic != FLOW_MAGIC) return fail(LBMP_ESTATE, "invalid flow handle");
    if (cls_host) LBMP_HIP(hipMemcpy(cls_host, f->d.cls, (size_t)f->N, hipMemcpyDeviceToHost));
    if (n_fluid) *n_fluid = f->nf;
    if (n_iface) *n_iface = f->ni;
    return LBMP_OK;
}

extern "C" void lb_flow_free(lbmp_flow* f) {
    if (f && f->magic == FLOW_MAGIC) {
        f->magic = 0;
        delete f;
    }
}
