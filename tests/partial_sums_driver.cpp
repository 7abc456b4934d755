// Blocks of the passes that write Gram sums of GMRES(3) steps, against the room of a region of
// partial sums (tests/test_partial_sums.py): every grid size, block cap, block height and
// batch size that a handle accepts. Host code only.
#include <cstdio>
#include <cstdlib>

#include "hm_gmres.hpp"

using namespace hm;

static int failures = 0, most = 0, most_product = 0;

static Grid grid(int n) {
    Grid g{};
    g.n = n;
    return g;
}

template <typename T>
static void check(const char* what, int n, int nblk) {
    if (gram_fits<T>(nblk) && nblk > 0) return;
    if (failures++ < 10) std::printf("%s: %d blocks on %d intervals\n", what, nblk, n);
}

template <typename T>
static void sizes(const LaunchCtx& ctx, int n) {
    const Grid g = grid(n);
    for (int nblk : {power_geom<StencilOp<T, 1>, T>(g, ctx).nblk, power_geom<StencilOp<T, 2>, T>(g, ctx).nblk,
                     power_geom<StencilOp<T, 3>, T>(g, ctx).nblk}) {
        check<T>("stored stencil", n, nblk);
        if (nblk > most) most = nblk;
    }
    const int product = power_geom<ProductOp<T, true>, T>(g, ctx).nblk;
    if (gram_fits<T>(product) && product > most_product) most_product = product;
}

template <typename T>
static void march(int n, int batch) {
    LaunchCtx ctx{};
    ctx.nrhs_cap = batch;
    const MarchShape m = march_shape<kMarchRows<T>>(n, batch, prereduce_blocks(ctx));
    check<T>("march", n, m.nblk);
    // the tiles cover the grid, and every tile has a wavefront
    if (m.strips * kMarchOwn < n + 1 || m.ntiles / m.strips * m.rows < n + 1 || m.nblk * kMarchWaves < m.ntiles ||
        m.nblk % 8 != 0)
        if (failures++ < 10) std::printf("march: %d intervals, batch %d not covered\n", n, batch);
    // one wavefront per SIMD with at most ten (FP32) or eight rows, else two and more
    const long long waves = (long long)m.ntiles * batch;
    if (batch == 1 && m.rows > 2 && waves > 8 * kComputeUnits) ++failures;
}

int main() {
    for (int n = 2; n <= 4096; ++n)
        for (int batch : {1, 2, 4, 9, 64, 4096}) {
            march<float>(n, batch);
            march<double>(n, batch);
        }
    for (int n = 1; n <= 2048; ++n)
        for (int batch : {1, 2, 9, 64})
            for (int cap : {64, 160, 320, 640, 1280, 7168})
                for (int tall : {4, 8, 16})
                    for (int small : {2, 4}) {
                        LaunchCtx ctx{};
                        ctx.nrhs = ctx.nrhs_cap = batch;
                        ctx.block_cap = cap;
                        ctx.tall_rows = tall;
                        ctx.small_rows = small;
                        sizes<float>(ctx, n);
                        sizes<double>(ctx, n);
                    }
    std::printf("at most %d blocks on stored stencils, %d on the product operator\n", most, most_product);
    return failures ? EXIT_FAILURE : EXIT_SUCCESS;
}
