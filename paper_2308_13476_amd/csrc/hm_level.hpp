// Shared by the level kernels: launch geometry, operator dispatch, and the
// tile-staged application of a level's operator.
#pragma once
#include <cstdlib>
#include <type_traits>
#include <utility>

#include <hip/hip_ext.h>

#include "hm_ops.hpp"

namespace hm {
namespace {

constexpr int kThreads = kBX * kBY;

// Block height: 64 x 4 for register-heavy Galerkin stencils; light kernels
// on grids of 256 or more intervals use ctx.tall_rows rows (4, 8 or 16), and
// grids of at most 128 intervals ctx.small_rows (2 or 4): their passes are
// latency-bound, and two wavefronts per block shorten each block's
// reductions and spread a pass over twice the compute units. Tiles keep an
// even first row, which the staging of the coarse grid correction relies on
// (it takes coarse row r0 / 2 as its reference). The handle's settings come
// from the environment at set-up or from the autotuner.
int block_rows(const Grid& g, bool heavy, const LaunchCtx& ctx) {
    if (g.n <= 128) return ctx.small_rows == 4 ? kBY : 2;
    if (heavy || g.n < 256) return kBY;
    return (ctx.tall_rows == 8 || ctx.tall_rows == 16) ? ctx.tall_rows : kBY;
}

// Rows per thread: enough that a level grid has at most `cap` blocks (the
// block cap of the context: every consumer of a reduction reads all partial
// sums of its producer, so more blocks cost more of those reads).
int level_rpt(const Grid& g, int by, int cap) {
    const long long m = g.n + 1;
    const long long bx = (m + kBX - 1) / kBX;
    const long long r = (m * bx + (long long)by * cap - 1) / ((long long)by * cap);
    return int(r < 1 ? 1 : r);
}

// Grid of a level launch. pad8 (handles for batches): the row-block count is
// raised until the tiles of one right-hand side are a multiple of 8, so that
// tile t of every right-hand side is dispatched to the same XCD (workgroups
// go to the eight XCDs round-robin by linear id) and the operator data all
// right-hand sides share (stencil coefficient planes, k^2) is fetched once
// into that XCD's L2 instead of once per right-hand side. The extra tiles lie
// below the grid: their blocks touch no node and write zero partial sums.
dim3 level_grid(const Grid& g, int rpt, int nrhs, int by, bool pad8 = false) {
    const unsigned gx = (g.n + 1 + kBX - 1) / kBX;
    unsigned gy = (g.n + 1 + by * rpt - 1) / (by * rpt);
    if (pad8)
        while ((gx * gy) % 8 != 0) ++gy;
    return dim3(gx, gy, nrhs);
}

struct Geom {
    int by, rpt, nblk;
    dim3 grid, block;
};

Geom geom(const Grid& g, bool heavy, const LaunchCtx& ctx) {
    Geom q;
    q.by = block_rows(g, heavy, ctx);
    q.rpt = level_rpt(g, q.by, ctx.block_cap);
    q.grid = level_grid(g, q.rpt, ctx.nrhs, q.by, ctx.nrhs_cap > 1);
    q.block = dim3(kBX, q.by);
    q.nblk = int(q.grid.x * q.grid.y);
    return q;
}

// Geometry of an operator kernel: the level geometry with rows per thread
// lowered until the block's LDS stages fit kMaxTileBytes.
constexpr size_t kMaxTileBytes = 64 * 1024;
template <typename Op, typename T>
__host__ __device__ size_t tile_bytes(int by, int rpt);
template <typename Op, typename T>
Geom geom_op(const Grid& g, const LaunchCtx& ctx) {
    Geom q = geom(g, Op::kHeavy, ctx);
    if (tile_bytes<Op, T>(q.by, q.rpt) > kMaxTileBytes) {
        while (q.rpt > 1 && tile_bytes<Op, T>(q.by, q.rpt) > kMaxTileBytes) --q.rpt;
        q.grid = level_grid(g, q.rpt, ctx.nrhs, q.by, ctx.nrhs_cap > 1);
        q.nblk = int(q.grid.x * q.grid.y);
    }
    return q;
}

// Calls f(integral_constant<int, BY>) for the runtime block height; kernels
// of register-heavy operators are only instantiated with short blocks.
template <bool kHeavy = false, typename F>
void with_by(int by, F&& f) {
    if (by == 2) {
        f(std::integral_constant<int, 2>{});
        return;
    }
    if constexpr (kHeavy) {
        f(std::integral_constant<int, kBY>{});
    } else {
        if (by == 16) f(std::integral_constant<int, 16>{});
        else if (by == 8) f(std::integral_constant<int, 8>{});
        else f(std::integral_constant<int, kBY>{});
    }
}

// Calls f(op) with the concrete operator type of the level.
template <typename T, typename F>
void with_op(const LevelOp<T>& lop, F&& f) {
    if (lop.level == 0) {
        f(FineOp<T>{lop.g, lop.k2, T(1.0 / (lop.h * lop.h)), T(2.0 / lop.h)});
        return;
    }
    if (lop.level == 1 && lop.product) {
        const FineOp<T> fine{lop.g0, lop.k2, T(1.0 / (lop.h * lop.h)), T(2.0 / lop.h)};
        const int D = 2 * lop.radius + 1;
        const cplx<T>* diagc = lop.coef + (long long)(lop.radius * D + lop.radius) * lop.g.plane;
        if (lop.transfer == 0) f(ProductOp<T, true>{lop.g, fine, T(lop.shift), diagc});
        else f(ProductOp<T, false>{lop.g, fine, T(lop.shift), diagc});
        return;
    }
    switch (lop.radius) {
        case 1: f(StencilOp<T, 1>{lop.g, lop.coef}); break;
        case 2: f(StencilOp<T, 2>{lop.g, lop.coef}); break;
        default: f(StencilOp<T, 3>{lop.g, lop.coef}); break;
    }
}

template <typename T>
__device__ __forceinline__ double dnorm2(cplx<T> z) {
    return double(z.re) * double(z.re) + double(z.im) * double(z.im);
}

// Stages 2-4 of a ProductOp apply, after the coarse tile (halo 3) is in LDS:
// y = P x and v = C_s y on the block's fine region, then the restriction of v
// at each coarse node, handed to f(i, j, p, pget(p), x at p, A_1 x at p).
template <typename T, bool kBez, typename PGet, typename F>
__device__ __forceinline__ void product_stages(const ProductOp<T, kBez>& op, const Tile<3>& tl, cplx<T>* lds,
                                               PGet&& pget, F&& f) {
    using PS = ProductStages<T>;
    if (tl.r0 > op.g.n) return;  // padding tile of a batch grid: no coarse node
    const int rows = tl.rows;
    cplx<T>* y = lds + Tile<3>::TW * (rows + 6);
    cplx<T>* v = y + PS::YW * PS::yrows(rows);
    const int nt = blockDim.x * blockDim.y;
    const int tid = threadIdx.y * kBX + threadIdx.x;
    const int nf = op.fine.g.n;
    const int fx0 = 2 * tl.c0 - 3, fy0 = 2 * tl.r0 - 3;  // fine origin of y
    // y = P x: even fine index 2K takes (1/8, 3/4, 1/8) of K-1, K, K+1 (Bezier)
    // or x_K (linear); odd 2K+1 takes (x_K + x_{K+1}) / 2. Zero off the fine
    // grid. One step forms the 2 x 2 fine nodes 2K + {0, 1}, 2L + {0, 1} from
    // the 3 x 3 coarse values around (K, L), rows first. K = c0 - 2 .. c0 + 64
    // and L = r0 - 2 .. r0 + rows cover y; the fine column and row 2 c0 - 4,
    // 2 r0 - 4 of the first steps lie outside it and are dropped.
    constexpr int PX = kBX + 3;
    const int np = PX * (rows + 3);
    const int ny = PS::yrows(rows);
    auto put = [&](int fi, int fj, cplx<T> val) {
        const int a = fi - fx0, bq = fj - fy0;
        if (a < 0 || bq < 0 || a >= PS::YW || bq >= ny) return;
        const bool in = fi >= 0 && fj >= 0 && fi <= nf && fj <= nf;
        y[bq * PS::YW + a] = in ? val : cplx<T>{T(0), T(0)};
    };
    for (int q = tid; q < np; q += nt) {
        const int K = tl.c0 - 2 + q % PX, L = tl.r0 - 2 + q / PX;
        const int base = tl.at(K - 1, L - 1);
        cplx<T> he[3], ho[3];  // rows L - 1 .. L + 1 at fine columns 2K, 2K + 1
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const cplx<T> xa = lds[base + t * Tile<3>::TW];
            const cplx<T> xb = lds[base + t * Tile<3>::TW + 1];
            const cplx<T> xc = lds[base + t * Tile<3>::TW + 2];
            if (kBez) {
                he[t].re = T(0.125) * xa.re + T(0.75) * xb.re + T(0.125) * xc.re;
                he[t].im = T(0.125) * xa.im + T(0.75) * xb.im + T(0.125) * xc.im;
            } else {
                he[t] = xb;
            }
            ho[t].re = T(0.5) * (xb.re + xc.re);
            ho[t].im = T(0.5) * (xb.im + xc.im);
        }
        cplx<T> e0, o0;  // fine row 2L
        if (kBez) {
            e0.re = T(0.125) * he[0].re + T(0.75) * he[1].re + T(0.125) * he[2].re;
            e0.im = T(0.125) * he[0].im + T(0.75) * he[1].im + T(0.125) * he[2].im;
            o0.re = T(0.125) * ho[0].re + T(0.75) * ho[1].re + T(0.125) * ho[2].re;
            o0.im = T(0.125) * ho[0].im + T(0.75) * ho[1].im + T(0.125) * ho[2].im;
        } else {
            e0 = he[1];
            o0 = ho[1];
        }
        put(2 * K, 2 * L, e0);
        put(2 * K + 1, 2 * L, o0);
        put(2 * K, 2 * L + 1, cplx<T>{T(0.5) * (he[1].re + he[2].re), T(0.5) * (he[1].im + he[2].im)});
        put(2 * K + 1, 2 * L + 1, cplx<T>{T(0.5) * (ho[1].re + ho[2].re), T(0.5) * (ho[1].im + ho[2].im)});
    }
    __syncthreads();
    // v = C_s y = A_s y - i beta2 W k^2 y on fine nodes of the grid, zero
    // elsewhere. One step takes the 2 x 2 fine nodes 2K + {0, 1}, 2L + {0, 1}
    // with their 12 distinct y neighbours, K = c0 - 1 .. c0 + 64 and
    // L = r0 - 1 .. r0 + rows; the last fine column and row of these steps lie
    // outside v and are dropped (their neighbours beyond y are read clamped).
    // k^2 of kVBlocks steps is loaded before their arithmetic (nodes off the
    // fine grid read a clamped in-grid node and give zero).
    constexpr int VX = kBX + 2;
    constexpr int kVBlocks = 2;
    const int nvb = VX * (rows + 2);
    T kk[kVBlocks][4];
    auto yat = [&](int c, int r) { return y[min(r, ny - 1) * PS::YW + min(c, PS::YW - 1)]; };
    auto cs_node = [&](int i, int j, T k2v, cplx<T> c, cplx<T> xw, cplx<T> xe, cplx<T> xs, cplx<T> xn) {
        cplx<T> r{T(0), T(0)};
        if (i >= 0 && j >= 0 && i <= nf && j <= nf) {
            r = op.fine.apply5k(i, j, k2v, c, xw, xe, xs, xn);
            const T sw = op.shift * line_w<T>(i, nf) * line_w<T>(j, nf) * k2v;
            r.re += sw * c.im;
            r.im -= sw * c.re;
        }
        return r;
    };
    // fine regions strictly inside the grid skip the boundary terms (a uniform
    // branch between two versions of the loop)
    const bool interior = 2 * tl.c0 - 2 >= 1 && 2 * tl.c0 + 2 * VX - 3 <= nf - 1 && 2 * tl.r0 - 2 >= 1 &&
                          2 * tl.r0 + 2 * rows + 1 <= nf - 1;
    auto cs_inner = [&](T k2v, cplx<T> c, cplx<T> xw, cplx<T> xe, cplx<T> xs, cplx<T> xn) {
        cplx<T> r = op.fine.apply5k_interior(k2v, c, xw, xe, xs, xn);
        const T sw = op.shift * k2v;
        r.re += sw * c.im;
        r.im -= sw * c.re;
        return r;
    };
    auto vstage = [&](auto inner) {
    for_strided_batched<kVBlocks>(
        nvb,
        [&](int u, int q) {
            const int fi = 2 * (tl.c0 - 1 + q % VX), fj = 2 * (tl.r0 - 1 + q / VX);
            const int i0 = min(max(fi, 0), nf), i1 = min(max(fi + 1, 0), nf);
            const int j0 = min(max(fj, 0), nf), j1 = min(max(fj + 1, 0), nf);
            kk[u][0] = op.fine.k2[op.fine.g.at(i0, j0)];
            kk[u][1] = op.fine.k2[op.fine.g.at(i1, j0)];
            kk[u][2] = op.fine.k2[op.fine.g.at(i0, j1)];
            kk[u][3] = op.fine.k2[op.fine.g.at(i1, j1)];
        },
        [&](int u, int q) {
            const int bx = q % VX, by = q / VX;
            const int fi = 2 * (tl.c0 - 1 + bx), fj = 2 * (tl.r0 - 1 + by);
            const int c = 2 * bx + 1, r = 2 * by + 1;  // y column and row of (fi, fj)
            const cplx<T> s0 = yat(c, r - 1), s1 = yat(c + 1, r - 1);
            const cplx<T> w0 = yat(c - 1, r), c00 = yat(c, r), c10 = yat(c + 1, r), e0 = yat(c + 2, r);
            const cplx<T> w1 = yat(c - 1, r + 1), c01 = yat(c, r + 1), c11 = yat(c + 1, r + 1), e1 = yat(c + 2, r + 1);
            const cplx<T> n0 = yat(c, r + 2), n1 = yat(c + 1, r + 2);
            const int vi = 2 * by * PS::VW + 2 * bx;
            const bool east = bx < VX - 1, north = by < rows + 1;
            if constexpr (decltype(inner)::value) {
                v[vi] = cs_inner(kk[u][0], c00, w0, c10, s0, c01);
                if (east) v[vi + 1] = cs_inner(kk[u][1], c10, c00, e0, s1, c11);
                if (north) {
                    v[vi + PS::VW] = cs_inner(kk[u][2], c01, w1, c11, c00, n0);
                    if (east) v[vi + PS::VW + 1] = cs_inner(kk[u][3], c11, c01, e1, c10, n1);
                }
            } else {
                v[vi] = cs_node(fi, fj, kk[u][0], c00, w0, c10, s0, c01);
                if (east) v[vi + 1] = cs_node(fi + 1, fj, kk[u][1], c10, c00, e0, s1, c11);
                if (north) {
                    v[vi + PS::VW] = cs_node(fi, fj + 1, kk[u][2], c01, w1, c11, c00, n0);
                    if (east) v[vi + PS::VW + 1] = cs_node(fi + 1, fj + 1, kk[u][3], c11, c01, e1, c10, n1);
                }
            }
        });
    };
    if (interior) vstage(std::true_type{});
    else vstage(std::false_type{});
    __syncthreads();
    // (R v)_I = (1/4) sum of the prolongation weights of I times v
    const T m5[5] = {T(1), T(4), T(6), T(4), T(1)};
    const T m3[5] = {T(0), T(1), T(2), T(1), T(0)};
    const T scale = kBez ? T(1.0 / 256.0) : T(1.0 / 16.0);
    constexpr int NB = 2;
    decltype(pget(0LL)) pv[NB];
    for_nodes_batched<NB>(op.g, (rows + blockDim.y - 1) / blockDim.y, [&](int u, long long p) { pv[u] = pget(p); },
                          [&](int u, int i, int j, long long p) {
        const int vc = (2 * (j - tl.r0) + 2) * PS::VW + 2 * (i - tl.c0) + 2;
        cplx<T> acc{T(0), T(0)};
#pragma unroll
        for (int dy = -2; dy <= 2; ++dy) {
            cplx<T> row{T(0), T(0)};
#pragma unroll
            for (int dx = -2; dx <= 2; ++dx) {
                const T w = kBez ? m5[dx + 2] : m3[dx + 2];
                const cplx<T> vv = v[vc + dy * PS::VW + dx];
                row.re += w * vv.re;
                row.im += w * vv.im;
            }
            const T w = kBez ? m5[dy + 2] : m3[dy + 2];
            acc.re += w * row.re;
            acc.im += w * row.im;
        }
        f(i, j, p, pv[u], lds[tl.at(i, j)], scale * acc);
    });
}

template <typename Op, typename T, typename PGet, typename F>
__device__ __forceinline__ void apply_from_tile(const Op& op, int rpt, const Tile<op_radius<Op>::value>& tl,
                                                cplx<T>* lds, PGet&& pget, F&& f);

// Runs f(i, j, p, pget(p), x at p, A x at p) over the thread's nodes, where
// x = xmake(xload(p)) (xload only loads): x for the block tile plus halo is
// staged in LDS first (one evaluation per tile node instead of one per
// stencil entry), then the operator reads LDS only. pget loads the caller's
// per-node operands; they and the operator's own (k^2 on level 0) are
// loaded for a batch of rows before the batch's arithmetic.
template <typename Op, typename T, typename XLoad, typename XMake, typename PGet, typename F>
__device__ __forceinline__ void for_nodes_applied_pre(const Op& op, int rpt, XLoad&& xload, XMake&& xmake,
                                                      PGet&& pget, F&& f) {
    constexpr int R = op_radius<Op>::value;
    cplx<T>* lds = reinterpret_cast<cplx<T>*>(hm_dyn_lds);
    const Tile<R> tl = block_tile<R>(rpt);
    fill_tile<T, R>(lds, tl, op.g, xload, xmake);
    apply_from_tile<Op, T>(op, rpt, tl, lds, pget, f);
}

// The second half of for_nodes_applied_pre: x of the block tile plus halo is
// in LDS (after a barrier); runs f(i, j, p, pget(p), x at p, A x at p).
template <typename Op, typename T, typename PGet, typename F>
__device__ __forceinline__ void apply_from_tile(const Op& op, int rpt, const Tile<op_radius<Op>::value>& tl,
                                                cplx<T>* lds, PGet&& pget, F&& f) {
    if constexpr (is_product<Op>::value) {
        product_stages(op, tl, lds, pget, f);
    } else if constexpr (std::is_same<Op, FineOp<T>>::value) {
        // tiles whose nodes all lie strictly inside the grid skip the boundary
        // terms (a uniform branch between two versions of the row loop)
        const int n = op.g.n;
        const bool interior = tl.c0 >= 1 && tl.c0 + kBX <= n && tl.r0 >= 1 && tl.r0 + tl.rows <= n;
        constexpr int NB = sizeof(T) == 4 ? 8 : 4;
        constexpr int TW = Tile<1>::TW;
        decltype(pget(0LL)) pv[NB];
        T kk[NB];
        auto rows = [&](auto inner) {
            for_nodes_batched<NB>(
                op.g, rpt,
                [&](int u, long long p) {
                    pv[u] = pget(p);
                    kk[u] = op.k2[p];
                },
                [&](int u, int i, int j, long long p) {
                    const int li = tl.at(i, j);
                    const cplx<T> c = lds[li];
                    const cplx<T> ax =
                        decltype(inner)::value
                            ? op.apply5k_interior(kk[u], c, lds[li - 1], lds[li + 1], lds[li - TW], lds[li + TW])
                            : op.apply5k(i, j, kk[u], c, lds[li - 1], lds[li + 1], lds[li - TW], lds[li + TW]);
                    f(i, j, p, pv[u], c, ax);
                });
        };
        if (interior) rows(std::true_type{});
        else rows(std::false_type{});
    } else {
        // rows per batch: stored stencils keep one row per thread on most
        // levels and their FP64 coefficient batches need the registers
        constexpr int NB = is_stencil<Op>::value ? (sizeof(T) == 4 ? 2 : 1) : (sizeof(T) == 4 ? 8 : 4);
        decltype(pget(0LL)) pv[NB];
        typename OpPre<Op>::type ov[NB];
        for_nodes_batched<NB>(
            op.g, rpt,
            [&](int u, long long p) {
                pv[u] = pget(p);
                ov[u] = OpPre<Op>::load(op, p);
            },
            [&](int u, int i, int j, long long p) {
                const int li = tl.at(i, j);
                f(i, j, p, pv[u], lds[li], apply_tile_pre(op, lds, li, i, j, p, ov[u]));
            });
    }
}

// for_nodes_applied_pre with x loaded as it is stored (xget(p) = x[p]) and
// no per-node operands of the caller: f(i, j, p, x at p, A x at p).
template <typename Op, typename T, typename XGet, typename F>
__device__ __forceinline__ void for_nodes_applied(const Op& op, int rpt, XGet&& xget, F&& f) {
    for_nodes_applied_pre<Op, T>(op, rpt, xget, Ident{}, [](long long) { return NoVals{}; },
                                 [&](int i, int j, long long p, NoVals, cplx<T> x, auto ax) { f(i, j, p, x, ax); });
}

// Dynamic LDS bytes of an operator kernel launched with geometry (by, rpt).
template <typename Op, typename T>
__host__ __device__ size_t tile_bytes(int by, int rpt) {
    constexpr int R = op_radius<Op>::value;
    if constexpr (is_product<Op>::value) return ProductStages<T>::values(by * rpt) * sizeof(cplx<T>);
    return size_t(Tile<R>::TW) * size_t(by * rpt + 2 * R) * sizeof(cplx<T>);
}

// Prolongation of §4 per dimension: fine 2I <- (e[I-1] + 6 e[I] + e[I+1]) / 8,
// fine 2I+1 <- (e[I] + e[I+1]) / 2 (linear transfer: fine 2I <- e[I]);
// coarse ghosts are zero, which drops out-of-range coarse indices.
template <typename T>
__device__ __forceinline__ void taps(int i, bool bez, T (&w)[3]) {
    if (i & 1) {
        w[0] = T(0); w[1] = T(0.5); w[2] = T(0.5);
    } else if (bez) {
        w[0] = T(0.125); w[1] = T(0.75); w[2] = T(0.125);
    } else {
        w[0] = T(0); w[1] = T(1); w[2] = T(0);
    }
}

// A powers pass launches at most this many blocks per right-hand side: every
// block of its consumers reads all of their partial sums.
constexpr int kPowMaxBlocks = 512;
constexpr int kComputeUnits = 256;

inline double* region(const LaunchCtx& ctx, int r) {
    return ctx.partials + (long long)r * ctx.nrhs_cap * kPartStride;
}

}  // namespace

#define HM_ACTIVE ctx.active

// Launches KERNEL<..., BY> with the geometry q (BY = q.by).
#define HM_LAUNCH(q, KERNEL_BY, ...)                                                                       \
    with_by((q).by, [&](auto byc) {                                                                        \
        constexpr int BY = decltype(byc)::value;                                                          \
        hipLaunchKernelGGL(KERNEL_BY, (q).grid, (q).block, 0, ctx.stream, __VA_ARGS__);                   \
    })
// Same for kernels templated on an operator type Op (heavy operators: short
// blocks only; Galerkin levels get their LDS tile as dynamic shared memory).
#define HM_LAUNCH_OP(q, KERNEL_BY, ...)                                                                    \
    with_by<Op::kHeavy>((q).by, [&](auto byc) {                                                            \
        constexpr int BY = decltype(byc)::value;                                                          \
        const size_t shm_ = tile_bytes<Op, T>((q).by, (q).rpt);                                           \
        hipLaunchKernelGGL(KERNEL_BY, (q).grid, (q).block, shm_, ctx.stream, __VA_ARGS__);                \
    })

}  // namespace hm
