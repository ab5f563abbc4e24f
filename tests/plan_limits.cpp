// Which step launches the library's rules (plan.hpp) take. Per line of input:
// variant K species_per_block quantities geometries {nx ny nz S nf nch gnh}...
// prints 1 where the launch is one the runtime takes, else 0.
#include <cstdio>

#include "plan.hpp"

int main() {
    int v, K, gs, nq, n;
    while (scanf("%d %d %d %d %d", &v, &K, &gs, &nq, &n) == 5) {
        std::vector<lbmp::PlanGeom> g(n);
        for (auto& p : g) {
            long long nf, nch;
            if (scanf("%d %d %d %d %lld %lld %d", &p.nx, &p.ny, &p.nz, &p.S, &nf, &nch, &p.gnh) != 7) return 1;
            p.nf = nf;
            p.nch = nch;
        }
        printf("%d\n", lbmp::plan_launchable(g.data(), n, v, K, gs, nq) ? 1 : 0);
    }
    return 0;
}
