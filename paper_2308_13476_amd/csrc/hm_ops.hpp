// Device operators of one level and the deterministic block reduction used
// by every kernel that produces norms or inner products.
#pragma once
#include "hm_common.hpp"
#include "hm_kernels.hpp"

namespace hm {

// Level 0: the scaled discrete operator A_s = W A of MP 2-A/2-B (§2),
// evaluated from k^2 on the fly. With edge weights w_e (1/2 for an edge that
// lies on the boundary, 1 otherwise) it reads
//   (A_s x)_p = W_p (4/h^2 - k_p^2 - 2 i k_p s_p / h) x_p
//               - (1/h^2) [ w_j (x_W + x_E) + w_i (x_S + x_N) ],
// where s_p counts the boundary sides of p; ghost nodes hold zero, which
// drops the couplings that the ghost elimination of the absorbing condition
// folded into the interior-normal neighbour (their weight 2 times W_p = 1/2
// is the edge weight 1).
template <typename T>
struct FineOp {
    static constexpr bool kHeavy = false;  // few registers: tall blocks
    Grid g;
    const T* k2;
    T ih2;    // 1 / h^2
    T two_h;  // 2 / h
    // diagonal at node (i, j) with k^2 = kk there
    __device__ __forceinline__ cplx<T> diag_k(int i, int j, T kk) const {
        const int n = g.n;
        const T W = line_w<T>(i, n) * line_w<T>(j, n);
        const int s = (i == 0 || i == n) + (j == 0 || j == n);
        T im = T(0);
        if (s) im = -two_h * T(s) * sqrt(kk);
        return {W * (T(4) * ih2 - kk), W * im};
    }
    __device__ __forceinline__ cplx<T> diag(int i, int j, long long p) const { return diag_k(i, j, k2[p]); }
    // (A_s x)_p from k^2 at p, the centre value and the west, east, south,
    // north neighbours
    __device__ __forceinline__ cplx<T> apply5k(int i, int j, T kk, cplx<T> c, cplx<T> xw, cplx<T> xe, cplx<T> xs,
                                               cplx<T> xn) const {
        const int n = g.n;
        const cplx<T> d = diag_k(i, j, kk);
        const T cx = ih2 * line_w<T>(j, n), cy = ih2 * line_w<T>(i, n);
        cplx<T> y = d * c;
        y.re -= cx * (xw.re + xe.re) + cy * (xs.re + xn.re);
        y.im -= cx * (xw.im + xe.im) + cy * (xs.im + xn.im);
        return y;
    }
    // the same at a node strictly inside the grid (W = 1, no Sommerfeld term):
    // equal to apply5k there, without the boundary arithmetic
    __device__ __forceinline__ cplx<T> apply5k_interior(T kk, cplx<T> c, cplx<T> xw, cplx<T> xe, cplx<T> xs,
                                                        cplx<T> xn) const {
        const T d = T(4) * ih2 - kk;
        cplx<T> y{d * c.re, d * c.im};
        y.re -= ih2 * (xw.re + xe.re) + ih2 * (xs.re + xn.re);
        y.im -= ih2 * (xw.im + xe.im) + ih2 * (xs.im + xn.im);
        return y;
    }
    __device__ __forceinline__ cplx<T> apply5(int i, int j, long long p, cplx<T> c, cplx<T> xw, cplx<T> xe,
                                              cplx<T> xs, cplx<T> xn) const {
        return apply5k(i, j, k2[p], c, xw, xe, xs, xn);
    }
    template <typename X>
    __device__ __forceinline__ cplx<T> apply_at(const X& x, int i, int j, long long p) const {
        return apply5(i, j, p, x(p), x(p - 1), x(p + 1), x(p - g.pitch), x(p + g.pitch));
    }
    __device__ __forceinline__ cplx<T> apply(const cplx<T>* __restrict__ x, int i, int j, long long p) const {
        return apply_at([x](long long q) { return x[q]; }, i, j, p);
    }
};

// Levels >= 1: stored Galerkin stencil (§3) of radius R, one complex plane per
// offset; ghost coefficients are zero. A Galerkin operator R C P with
// R = P^T / 4 (§4) and a complex symmetric C (the scaled operator W A and its
// shifted form differ from their transposes in no entry) is complex
// symmetric: the coefficient of offset d at node p equals that of offset -d
// at node p + d, up to the rounding of the product that formed them. Passes
// read the offsets of the upper half (dy > 0, or dy = 0 and dx >= 0) at p and
// those of the lower half from the upper-half plane at p + d, so that only
// the upper half of the planes is streamed from memory (the mirrored reads
// are the neighbouring nodes' own coefficients, found in cache); the operator
// applied is then exactly symmetric.
template <typename T, int R>
struct StencilOp {
    static constexpr bool kHeavy = R >= 2;  // 25/49-point stencils: many registers, short blocks
    Grid g;
    const cplx<T>* __restrict__ coef;
    static constexpr int D = 2 * R + 1;
    __device__ __forceinline__ cplx<T> diag(int, int, long long p) const { return coef[(R * D + R) * g.plane + p]; }
    // coefficient of offset (dx, dy) at node p (dx, dy compile-time after unrolling)
    __device__ __forceinline__ cplx<T> at(int dy, int dx, long long p) const {
        const bool lower = dy < 0 || (dy == 0 && dx < 0);
        return lower ? coef[((R - dy) * D + R - dx) * g.plane + p + (long long)dy * g.pitch + dx]
                     : coef[((dy + R) * D + dx + R) * g.plane + p];
    }
    template <typename X>
    __device__ __forceinline__ cplx<T> apply_at(const X& x, int, int, long long p) const {
        cplx<T> y{T(0), T(0)};
#pragma unroll
        for (int dy = -R; dy <= R; ++dy)
#pragma unroll
            for (int dx = -R; dx <= R; ++dx) y = cfma(y, at(dy, dx, p), x(p + (long long)dy * g.pitch + dx));
        return y;
    }
    __device__ __forceinline__ cplx<T> apply(const cplx<T>* __restrict__ x, int i, int j, long long p) const {
        return apply_at([x](long long q) { return x[q]; }, i, j, p);
    }
};

// Level 1 without its stored stencil: A_1 = R C_s P (§3 Galerkin product, §4
// transfers) applied in three steps from level-0 data, y = P x on the fine
// grid, v = C_s y with the shifted Laplacian C_s = A_s - i beta2 W K^2 of
// level 0, then the restriction R = P^T / 4 of v. Equal to the stored
// Galerkin stencil up to rounding; reads x and level-0 k^2 instead of
// (2r+1)^2 complex coefficients per node. The Jacobi diagonal comes from the
// centre plane of the stored stencil.
template <typename T, bool kBez>
struct ProductOp {
    static constexpr bool kHeavy = true;  // short blocks: three LDS stages
    Grid g;                 // level 1
    FineOp<T> fine;         // level-0 operator A_s (grid, k^2, 1/h^2, 2/h)
    T shift;                // beta2
    const cplx<T>* diagc;   // centre plane of the stored level-1 stencil
    __device__ __forceinline__ cplx<T> diag(int, int, long long p) const { return diagc[p]; }
};

// Tile (column block, row block) of this workgroup: blockIdx.x, blockIdx.y.
// (A map that gave each XCD a contiguous run of tiles cut the halo re-reads
// between L2s but made the cycle slower, so tiles follow the block ids.)
struct BlockXY {
    int x, y;
};
__device__ __forceinline__ BlockXY block_xy() { return BlockXY{int(blockIdx.x), int(blockIdx.y)}; }

// Calls f(i, j, p) for the nodes of this thread: column bx * 64 + lane,
// rows interleaved by 4 over rows_per_thread consecutive row groups of row
// block by ((bx, by) = block_xy()).
template <typename F>
__device__ __forceinline__ void for_nodes(const Grid& g, int rpt, F&& f) {
    const BlockXY bt = block_xy();
    const int i = bt.x * kBX + threadIdx.x;
    if (i > g.n) return;
    const int by = blockDim.y;
    for (int rr = 0; rr < rpt; ++rr) {
        const int j = (bt.y * rpt + rr) * by + threadIdx.y;
        if (j > g.n) return;
        f(i, j, g.at(i, j));
    }
}

// Waits until every vector memory operation the wave has issued is done
// (s_waitcnt vmcnt(0); expcnt and lgkmcnt fields at their no-wait maxima).
// Placed after a sweep of loads so that the stores of the following
// arithmetic do not make the compiler wait for them row by row.
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// The nodes of for_nodes, taken NB rows at a time in two sweeps: load(u, p)
// for the rows of the batch first, then body(u, i, j, p) for the rows that
// exist. The loads of a batch are in flight together: one memory round trip
// per batch instead of one per row. Only the row count decides which loads
// are issued (uniform in the block, so no divergent branch separates them);
// a row below the grid loads its column's last node instead. kLoaded: the loads of
// the first batch were issued by first_node_loads, earlier in the kernel.
template <int NB, bool kLoaded = false, typename Load, typename Body>
__device__ __forceinline__ void for_nodes_batched(const Grid& g, int rpt, Load&& load, Body&& body) {
    const BlockXY bt = block_xy();
    const int i = bt.x * kBX + threadIdx.x;
    if (i > g.n) return;
    const int by = blockDim.y;
    const int j0 = bt.y * rpt * by + threadIdx.y;
    if (j0 > g.n) return;
    for (int rr0 = 0; rr0 < rpt; rr0 += NB) {
        if (!kLoaded || rr0 > 0)
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (rr0 + u < rpt) load(u, g.at(i, min(j0 + (rr0 + u) * by, g.n)));
        wait_vmem();
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int j = j0 + (rr0 + u) * by;
            if (rr0 + u < rpt && j <= g.n) body(u, i, j, g.at(i, j));
        }
    }
}

// The loads of the first batch of for_nodes_batched<NB, true> (threads
// without nodes load clamped ones).
template <int NB, typename Load>
__device__ __forceinline__ void first_node_loads(const Grid& g, int rpt, Load&& load) {
    const BlockXY bt = block_xy();
    const int i = min(bt.x * kBX + int(threadIdx.x), g.n), by = blockDim.y, j0 = bt.y * rpt * by + threadIdx.y;
#pragma unroll
    for (int u = 0; u < NB; ++u)
        if (u < rpt) load(u, g.at(i, min(j0 + u * by, g.n)));
}

// Indices q = tid, tid + nt, ... < count of a block-strided loop, NB at a
// time in two sweeps as in for_nodes_batched: load(u, q) (q clamped to
// count - 1 in the last, partly filled stride; strides beyond it are not
// loaded), then body(u, q) for the indices that exist. kLoaded: the first round's
// loads were issued by first_strided_loads.
template <int NB, typename Load>
__device__ __forceinline__ void first_strided_loads(int count, Load&& load) {
    const int nt = blockDim.x * blockDim.y;
    const int tid = threadIdx.y * kBX + threadIdx.x;
#pragma unroll
    for (int u = 0; u < NB; ++u)
        if (u * nt < count) load(u, min(tid + u * nt, count - 1));
}
template <int NB, bool kLoaded = false, typename Load, typename Body>
__device__ __forceinline__ void for_strided_batched(int count, Load&& load, Body&& body) {
    const int nt = blockDim.x * blockDim.y;
    const int tid = threadIdx.y * kBX + threadIdx.x;
    for (int s0 = 0; s0 < count; s0 += NB * nt) {  // uniform: first index of the round
        const int q0 = s0 + tid;
        if (!kLoaded || s0 > 0)
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (s0 + u * nt < count) load(u, min(q0 + u * nt, count - 1));
        wait_vmem();
#pragma unroll
        for (int u = 0; u < NB; ++u)
            if (q0 + u * nt < count) body(u, q0 + u * nt);
    }
}

// ---------------------------------------------------------------- LDS tiles
// A block of 64 x BY threads with rows_per_thread rpt covers columns
// [c0, c0 + 64) and rows [r0, r0 + BY * rpt) of a level. Its LDS tile adds a
// halo of R nodes on every side so that a radius-R stencil reads LDS only.
extern __shared__ __align__(16) unsigned char hm_dyn_lds[];

template <int R, int TX = kBX>
struct Tile {
    static constexpr int TW = TX + 2 * R;
    int c0, r0, rows;
    __device__ __forceinline__ int at(int i, int j) const { return (j - r0 + R) * TW + (i - c0 + R); }
    __device__ __forceinline__ int count() const { return TW * (rows + 2 * R); }
};

template <int R>
__device__ __forceinline__ Tile<R> block_tile(int rpt) {
    const BlockXY bt = block_xy();
    return Tile<R>{bt.x * kBX, bt.y * int(blockDim.y) * rpt, int(blockDim.y) * rpt};
}

// lds[t.at(i, j)] = make(load(g.at(i, j))) for every tile node inside the
// padded frame (ghosts read as stored, zero); nodes beyond it hold zero and
// are never used by an in-domain stencil. load only gathers the values that
// make combines: the loads of FillBatch<T> nodes are issued before any
// combination (a node outside the frame is clamped onto it, R <= kGhost, and
// gives zero), so that they are in flight together.
template <typename T>
struct FillBatch {
    static constexpr int value = sizeof(T) == 4 ? 8 : 4;  // register budget of FP64 tiles
};
struct Ident {
    template <typename X>
    __device__ __forceinline__ X operator()(const X& x) const { return x; }
};
template <typename T, int R>
__device__ __forceinline__ bool tile_below_grid(const Tile<R>& t, const Grid& g) {
    return t.r0 - R > g.n;  // padding tiles of batch grids (uniform in the block)
}
template <typename T, int R, typename Load, typename Make>
__device__ __forceinline__ void fill_tile(cplx<T>* lds, const Tile<R>& t, const Grid& g, Load&& load, Make&& make) {
    static_assert(R <= kGhost, "tile halo beyond the stored ghost layers");
    if (tile_below_grid<T, R>(t, g)) return;  // no node of the tile or its halo exists
    constexpr int FB = FillBatch<T>::value;
    decltype(load(0LL)) v[FB];
    bool ok[FB];
    for_strided_batched<FB>(
        t.count(),
        [&](int u, int q) {
            const int i = t.c0 - R + q % Tile<R>::TW;
            const int j = t.r0 - R + q / Tile<R>::TW;
            const int ic = min(max(i, -R), g.n + R), jc = min(max(j, -R), g.n + R);
            ok[u] = i == ic && j == jc;
            v[u] = load(g.at(ic, jc));
        },
        [&](int u, int q) { lds[q] = ok[u] ? make(v[u]) : cplx<T>{T(0), T(0)}; });
    __syncthreads();
}

// Stencil of radius R applied at node p whose tile index is li, values from LDS.
template <typename T, int R>
__device__ __forceinline__ cplx<T> apply_tile(const StencilOp<T, R>& op, const cplx<T>* lds, int li, long long p) {
    constexpr int TW = Tile<R>::TW;
    cplx<T> y{T(0), T(0)};
#pragma unroll
    for (int dy = -R; dy <= R; ++dy)
#pragma unroll
        for (int dx = -R; dx <= R; ++dx)
            y = cfma(y, op.at(dy, dx, p), lds[li + dy * TW + dx]);
    return y;
}

// Level-0 operator applied at tile index li from LDS, with k^2 at p given.
template <typename T>
__device__ __forceinline__ cplx<T> apply_tile(const FineOp<T>& op, const cplx<T>* lds, int li, int i, int j, T kk) {
    constexpr int TW = Tile<1>::TW;
    return op.apply5k(i, j, kk, lds[li], lds[li - 1], lds[li + 1], lds[li - TW], lds[li + TW]);
}

// Per-node operand of an operator that a batched sweep loads ahead of the
// arithmetic: k^2 for the level-0 operator; nothing for stored stencils,
// whose coefficient loads stay in the apply (one row per thread there).
struct NoVals {};
template <typename T, int N>
struct Vals {
    cplx<T> v[N];
};
template <typename Op>
struct OpPre {
    using type = NoVals;
    __device__ __forceinline__ static NoVals load(const Op&, long long) { return {}; }
};
template <typename T>
struct OpPre<FineOp<T>> {
    using type = T;
    __device__ __forceinline__ static T load(const FineOp<T>& op, long long p) { return op.k2[p]; }
};
template <typename T, int R>
__device__ __forceinline__ cplx<T> apply_tile_pre(const StencilOp<T, R>& op, const cplx<T>* lds, int li, int,
                                                  int, long long p, NoVals) {
    return apply_tile(op, lds, li, p);
}
template <typename T>
__device__ __forceinline__ cplx<T> apply_tile_pre(const FineOp<T>& op, const cplx<T>* lds, int li, int i, int j,
                                                  long long, T kk) {
    return apply_tile(op, lds, li, i, j, kk);
}

// sum_d c[d] x_d over N stencil entries that the thread holds in registers, at(d)
// reading x_d from LDS. The reads go out in batches of CH, each while the batch
// before it is multiplied: left to itself the compiler reads two values, waits and
// multiplies, 28 LDS round trips and 2800 cycles per radius-3 application whose
// multiply-adds take 800. Longer batches than the registers beside the stencil
// hold spill it. The additions keep the order of d.
template <typename T>
__device__ __forceinline__ void stay_here(cplx<T>& y) {  // reads above and sums below it keep their places
    __asm__ volatile("" : "+v"(y.re), "+v"(y.im)::"memory");
}
template <typename T, int N, int CH, typename At>
__device__ __forceinline__ cplx<T> held_sum(const cplx<T> (&c)[N], At&& at) {
    constexpr int NB = (N + CH - 1) / CH;
    cplx<T> v[2][CH];
    cplx<T> y{T(0), T(0)};
#pragma unroll
    for (int d = 0; d < CH && d < N; ++d) v[0][d] = at(d);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int d = 0; d < CH; ++d)
            if ((b + 1) * CH + d < N) v[(b + 1) & 1][d] = at((b + 1) * CH + d);
        stay_here(y);
#pragma unroll
        for (int d = 0; d < CH; ++d)
            if (b * CH + d < N) y = cfma(y, c[b * CH + d], v[b & 1][d]);
        stay_here(y);
    }
    return y;
}

// The same sum with less rounding (the Krylov vectors of FP32 steps, hm_gram.hpp): runs
// of kWideRun products are added up in FP32, the runs in FP64. Against sums in FP32 it
// costs 22.6 us (20.9) on 512 intervals, radius 2, and 20.8 (19.6), 9.9 (9.8), 8.2 (8.0) on
// 256, 128 and 64, radius 3. All in FP64, four conversions an entry, 26.6, 83 (spills),
// 11.5 and 9.9 for errors a fifth smaller; runs of a stencil's row are a tenth off.
constexpr int kWideRun = 3;
struct WideSum {
    cplx<double> y{0.0, 0.0};
    cplx<float> s{0.0f, 0.0f};
    // entry d of n (compile-time after unrolling)
    __device__ __forceinline__ void add(int d, int n, cplx<float> c, cplx<float> x) {
        s = d % kWideRun == 0 ? cplx<float>{fmaf(c.re, x.re, -(c.im * x.im)), fmaf(c.re, x.im, c.im * x.re)} : cfma(s, c, x);
        if (d % kWideRun == kWideRun - 1 || d == n - 1) y = y + cast<double>(s);
    }
};
template <int N, int CH, typename At>
__device__ __forceinline__ cplx<double> held_sum_wide(const cplx<float> (&c)[N], At&& at) {
    constexpr int NB = (N + CH - 1) / CH;
    cplx<float> v[2][CH];
    WideSum t;
#pragma unroll
    for (int d = 0; d < CH && d < N; ++d) v[0][d] = at(d);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int d = 0; d < CH; ++d)
            if ((b + 1) * CH + d < N) v[(b + 1) & 1][d] = at((b + 1) * CH + d);
        stay_here(t.s);
        stay_here(t.y);
#pragma unroll
        for (int d = 0; d < CH; ++d)
            if (b * CH + d < N) t.add(b * CH + d, N, c[b * CH + d], v[b & 1][d]);
        stay_here(t.s);
        stay_here(t.y);
    }
    return t.y;
}
template <int N, int CH, typename At>
__device__ __forceinline__ cplx<double> held_sum_wide(const cplx<double> (&c)[N], At&& at) {
    return held_sum<double, N, CH>(c, at);
}

template <typename Op>
struct is_stencil {
    static constexpr bool value = false;
};
template <typename T, int R>
struct is_stencil<StencilOp<T, R>> {
    static constexpr bool value = true;
    static constexpr int radius = R;
};

// Halo width of an operator's LDS tile.
template <typename Op>
struct op_radius {
    static constexpr int value = 1;  // level-0 five-point operator
};
template <typename T, int R>
struct op_radius<StencilOp<T, R>> {
    static constexpr int value = R;
};
// A stored FP32 stencil applied as in held_sum_wide.
template <int R>
struct WideStencil : StencilOp<float, R> {};
template <int R>
struct op_radius<WideStencil<R>> {
    static constexpr int value = R;
};
template <int R>
struct is_stencil<WideStencil<R>> {
    static constexpr bool value = true;
    static constexpr int radius = R;
};
template <int R>
__device__ __forceinline__ cplx<double> apply_tile_pre(const WideStencil<R>& op, const cplx<float>* lds, int li, int,
                                                       int, long long p, NoVals) {
    constexpr int TW = Tile<R>::TW;
    constexpr int D = 2 * R + 1;
    WideSum t;
#pragma unroll
    for (int d = 0; d < D * D; ++d)
        t.add(d, D * D, op.at(d / D - R, d % D - R, p), lds[li + (d / D - R) * TW + d % D - R]);
    return t.y;
}
template <typename Op>
__device__ __forceinline__ const Op& widened(const Op& op) { return op; }
template <int R>
__device__ __forceinline__ WideStencil<R> widened(const StencilOp<float, R>& op) { return WideStencil<R>{op}; }

template <typename T, bool B>
struct op_radius<ProductOp<T, B>> {
    static constexpr int value = 3;  // coarse halo that the fine stages need
};
template <typename Op>
struct is_product {
    static constexpr bool value = false;
};
template <typename T, bool B>
struct is_product<ProductOp<T, B>> {
    static constexpr bool value = true;
};

// Fine-grid stages of a ProductOp block. The block's coarse tile covers
// columns [c0, c0 + 64) and rows [r0, r0 + rows); the restriction reads fine
// nodes 2I - 2 .. 2I + 2, C_s one more on each side.
template <typename T>
struct ProductStages {
    static constexpr int YW = 2 * kBX + 5;  // fine columns 2 c0 - 3 .. 2 c0 + 129 (y = P x)
    static constexpr int VW = 2 * kBX + 3;  // fine columns 2 c0 - 2 .. 2 c0 + 128 (v = C_s y)
    __host__ __device__ static int yrows(int rows) { return 2 * rows + 5; }
    __host__ __device__ static int vrows(int rows) { return 2 * rows + 3; }
    __host__ __device__ static size_t values(int rows) {
        return size_t(Tile<3>::TW) * (rows + 6) + size_t(YW) * yrows(rows) + size_t(VW) * vrows(rows);
    }
};

__device__ __forceinline__ bool rhs_active(const int* active, int b) { return active == nullptr || active[b] != 0; }

// Grid-wide reductions without atomics. A producer kernel writes one partial
// sum per block (`block_partials`); the kernel launched after it reduces all
// partials itself (`reduce_partials`, identical order in every block, hence
// deterministic), the kernel boundary making the partials visible. The
// partials of right-hand side b and region r live at
// partials + (r * nrhs_cap + b) * kPartStride.

// Row-major index of this block's tile, the slot of its partial sums.
__device__ __forceinline__ int block_linear() {
    const BlockXY bt = block_xy();
    return bt.y * int(gridDim.x) + bt.x;
}
__device__ __forceinline__ int thread_linear() { return threadIdx.y * kBX + threadIdx.x; }

// Sum over the 64 lanes of a wavefront by DPP lane moves (no LDS traffic):
// pairwise within quads, rotations by 4 and 8 within rows of 16, then the
// sums of rows 0 and 2 broadcast into rows 1 and 3 and of rows 0-1 into rows
// 2-3. Lane 63 ends with the total; the order of the additions is fixed, so
// the result is deterministic. Doubles move as two 32-bit halves.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double x) {
    const unsigned long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, int(unsigned(b & 0xffffffffu)), CTRL, ROW_MASK, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, int(unsigned(b >> 32)), CTRL, ROW_MASK, 0xF, true);
    return __longlong_as_double((unsigned long long)unsigned(lo) | ((unsigned long long)unsigned(hi) << 32));
}

// One value summed over the 64 lanes of a wavefront by the moves of
// block_sum; lane 63 ends with the total.
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp_move<0xb1, 0xF>(x);
    x += dpp_move<0x4e, 0xF>(x);
    x += dpp_move<0x124, 0xF>(x);
    x += dpp_move<0x128, 0xF>(x);
    x += dpp_move<0x142, 0xA>(x);
    x += dpp_move<0x143, 0xC>(x);
    return x;
}

// Block sum for 64 x BY thread blocks, BY <= kMaxBY (wavefront = threadIdx.y):
// each wavefront reduces its K values with DPP moves, lane 63 stores them,
// and every thread adds the wavefront totals in wavefront order.
template <int K>
__device__ __forceinline__ void block_sum(double (&v)[K], double (&tot)[K]) {
    __shared__ double sh[kMaxBY][K];
    const int lane = threadIdx.x, wave = threadIdx.y;
    __syncthreads();  // sh may still be read from an earlier call
    double w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] = v[k];
    // the K values of one step are independent: their moves overlap
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] += dpp_move<0xb1, 0xF>(w[k]);  // quad_perm [1,0,3,2]
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] += dpp_move<0x4e, 0xF>(w[k]);  // quad_perm [2,3,0,1]
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] += dpp_move<0x124, 0xF>(w[k]);  // row_ror 4
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] += dpp_move<0x128, 0xF>(w[k]);  // row_ror 8
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] += dpp_move<0x142, 0xA>(w[k]);  // row_bcast 15 into rows 1, 3
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] += dpp_move<0x143, 0xC>(w[k]);  // row_bcast 31 into rows 2, 3
    if (lane == kBX - 1)
#pragma unroll
        for (int k = 0; k < K; ++k) sh[wave][k] = w[k];
    __syncthreads();
    // only the block's own wavefronts (a loop over every possible one with a
    // guard per term costs two selects and an add per term and wavefront)
    const int nw = blockDim.y;
#pragma unroll
    for (int k = 0; k < K; ++k) tot[k] = 0.0;
    for (int q = 0; q < nw; ++q)
#pragma unroll
        for (int k = 0; k < K; ++k) tot[k] += sh[q][k];
}

// Writes this block's K sums to out[block * K + k].
template <int K>
__device__ __forceinline__ void block_partials(double (&v)[K], double* out) {
    double tot[K];
    block_sum<K>(v, tot);
    if (thread_linear() == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) out[block_linear() * K + k] = tot[k];
    }
}

// Sums the K partials of nblk producer blocks; every thread gets the totals.
// Each thread sums partials q = tid, tid + nt, ... in that order; loads are
// gathered kReduceBatch strides at a time so that they are in flight together.
constexpr int kReduceBatch = 4;
template <int K>
__device__ __forceinline__ void reduce_partials(const double* in, int nblk, double (&tot)[K]) {
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    const int nt = blockDim.x * blockDim.y;
    for (int q0 = thread_linear(); q0 < nblk; q0 += kReduceBatch * nt) {
        double v[kReduceBatch][K];
#pragma unroll
        for (int u = 0; u < kReduceBatch; ++u) {
            const int q = q0 + u * nt;
#pragma unroll
            for (int k = 0; k < K; ++k) v[u][k] = (q < nblk) ? in[q * K + k] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kReduceBatch; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] += v[u][k];
    }
    block_sum<K>(acc, tot);
}

// 1 / x for x > 0 in FP64: the hardware estimate refined by two Newton steps
// (its relative error squares per step, ending at about one unit in the last
// place). It stands in for the correctly rounded division in the short dependent
// chain of the Gram elimination.
__device__ __forceinline__ double rcp_nr(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    y = fma(fma(-x, y, 1.0), y, y);
    return y;
}

}  // namespace hm
