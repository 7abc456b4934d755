// Coarse tail of the cycle: one workgroup per right-hand side runs the whole
// sub-cycle (§3 coarse grid correction, §5 V/W cycles) on the small levels at
// the bottom of the hierarchy. Every vector of those levels lives in LDS for
// the whole sub-cycle; barriers and block reductions replace the kernel
// launches and grid-wide reductions of the level kernels, which on grids of at
// most 17 x 17 nodes cost far more than the arithmetic.
//
// What bounds it is the latency of one compute unit: a chain of operator
// applications, each a barrier and a sweep of LDS reads away from the next. So
// two lanes share every node of a level: each loads half of the node's stencil
// into registers once per smoothing step (once per visit with Jacobi sweeps), an
// application reads LDS only, in batches that overlap the multiply-adds
// (held_sum), and GMRES(3) steps take one block reduction each (hm_gram.hpp).
// Levels 16, 8 and 4 of a V(1,1) cycle on 1024 intervals: 32.7 us in FP32 and 46.6 us in
// FP64, W(1,1) in FP32 on 512 intervals 44.0 us (41.7 and 49.7 on the first grid, 58 on
// the second with a whole stencil per thread and reads the compiler waits for two by
// two).
#include "hm_gram.hpp"

namespace hm {
namespace {

// Ten wavefronts: two lanes for each of the 289 nodes of a 16-interval level.
constexpr int kTailWaves = kTailThreads / 64;

// One level of the tail: its stencil in global memory and its LDS planes.
// LDS planes have a zero frame of kTailGhost nodes: node (i, j) sits at
// (j + kTailGhost) * lp + i + kTailGhost.
template <typename T>
struct TLv {
    Grid g;  // global layout (coefficient planes)
    const cplx<T>* coef;
    int m, lp, N;
    unsigned per_row;
    double sigma;
    cplx<T>* pl;  // planes: u, f, then r, v_1, v_2, v_3 on smoothed levels
    __device__ __forceinline__ cplx<T>* u() const { return pl; }
    __device__ __forceinline__ cplx<T>* f() const { return pl + lp * lp; }
    __device__ __forceinline__ cplx<T>* s(int k) const { return pl + (2 + k) * lp * lp; }
    __device__ __forceinline__ int row(int q) const { return int(unsigned(q) * per_row >> 16); }
    __device__ __forceinline__ int col(int q, int row) const { return q - row * m; }
    __device__ __forceinline__ int li(int q) const {
        const int j = row(q);
        return (j + kTailGhost) * lp + col(q, j) + kTailGhost;
    }
    __device__ __forceinline__ long long gi(int q) const {
        const int j = row(q);
        return g.at(col(q, j), j);
    }
};

template <typename T>
__device__ __forceinline__ TLv<T> tail_level(const TailArgs<T>& a, int q, cplx<T>* lds) {
    TLv<T> v;
    v.g = a.lv[q].g;
    v.m = v.g.n + 1;
    v.N = v.m * v.m;
    v.lp = tail_pitch(v.g.n);
    v.coef = a.lv[q].coef;
    v.sigma = a.lv[q].sigma;
    v.per_row = a.lv[q].per_row;
    v.pl = lds + a.lv[q].off;
    return v;
}

// f(q) for the nodes of a level, a thread per node (in turns on levels of more
// than kTailThreads nodes).
template <typename T, typename F>
__device__ __forceinline__ void tnodes(const TLv<T>& L, F&& f) {
    for (int q = thread_here(); q < L.N; q += kTailThreads) f(q);
}

// The stencil of a node in the registers of two lanes (levels of at most
// kTailThreads / 2 nodes): lanes l and l + 32 of a wavefront hold node
// 32 wave + l, lanes below 32 the centre, the rows above it and the middle row up to
// the centre, the others a zero, the rows below and the rest of the middle row.
// Lanes without a node hold the stencil of node 0 and take no part.
__device__ __forceinline__ int held_node() {
    const int t = thread_here();
    return (t >> 6) * 32 + (t & 31);
}
__device__ __forceinline__ int held_part() { return (thread_here() >> 5) & 1; }
template <typename T, int R>
struct THeld {
    static constexpr int kRadius = R, D = 2 * R + 1;
    static constexpr int kTaps = R * D + R + 1;
    static constexpr bool kHeld = true;
    cplx<T> c[kTaps];
    __device__ __forceinline__ void load(const TLv<T>& L) {
        // uniform plane bases plus one 32-bit offset, made here each time:
        // addresses kept in registers by the compiler spilled the stencil
        const unsigned pb = unsigned(L.g.plane) * unsigned(sizeof(cplx<T>)), part = held_part();
        const int q = held_node();
        const unsigned off = unsigned(L.gi(q < L.N ? q : 0)) * unsigned(sizeof(cplx<T>));
        unsigned rows = off + part * (R + 1) * D * pb, mid = off + (R * D + part * (R + 1)) * pb;
        __asm__ volatile("" : "+v"(rows), "+v"(mid));
        const char* base = reinterpret_cast<const char*>(L.coef);
#pragma unroll
        for (int d = 0; d < R * D; ++d) c[1 + d] = *reinterpret_cast<const cplx<T>*>(base + (long long)d * pb + rows);
#pragma unroll
        for (int d = 0; d < R; ++d)
            c[1 + R * D + d] = *reinterpret_cast<const cplx<T>*>(base + (long long)d * pb + mid);
        c[0] = cplx<T>{T(0), T(0)};
        if (part == 0) c[0] = *reinterpret_cast<const cplx<T>*>(base + (long long)R * pb + mid);
    }
    // (A x)_q at the LDS index ln of the node, in both of its lanes (wide: FP64, summed as
    // in held_sum_wide).
    template <bool kWide = false>
    __device__ __forceinline__ auto apply(const TLv<T>& L, int ln, const cplx<T>* x) const {
        const int part = held_part();
        const cplx<T>* rows = x + ln + (part ? 1 : -R) * L.lp - R;
        const cplx<T>* mid = x + ln + (part ? 1 : -R);
        const cplx<T>* first = x + ln + (part ? R : 0);  // beside the zero: any node of the middle row
        auto at = [&](int d) {
            return d == 0 ? *first : (d - 1 < R * D ? rows[(d - 1) / D * L.lp + (d - 1) % D] : mid[d - 1 - R * D]);
        };
        constexpr int CH = sizeof(T) == 4 ? 9 : 4;
        if constexpr (kWide) {
            const cplx<double> y = held_sum_wide<kTaps, CH>(c, at);
            return cplx<double>{half_sum(y.re), half_sum(y.im)};
        } else {
            const cplx<T> y = held_sum<T, kTaps, CH>(c, at);
            return cplx<T>{half_sum(y.re), half_sum(y.im)};
        }
    }
};
// Larger levels: threads take nodes in turns, coefficients from memory.
template <int R>
struct TBig {
    static constexpr int kRadius = R;
    static constexpr bool kHeld = false;
    template <typename T>
    __device__ __forceinline__ void load(const TLv<T>&) {}
};
template <typename H>
struct TTag {
    using type = H;
};
constexpr int kBigNodes = kTailNodesPerThread;

// out(l, (A x)_q) for every node, l its LDS index (ln: that of the held node of
// this lane, or -1), x a plane of the level. kInPlace: out may overwrite x, so
// every thread reads x before any out. Ends with a barrier.
template <bool kInPlace, typename T, int R, typename F>
__device__ __forceinline__ void tail_apply(const TLv<T>& L, int ln, const THeld<T, R>& h, const cplx<T>* x, F&& out) {
    cplx<T> y{T(0), T(0)};
    if (ln >= 0) y = h.apply(L, ln, x);
    if constexpr (kInPlace) __syncthreads();
    if (ln >= 0 && held_part() == 0) out(ln, y);
    __syncthreads();
}
template <bool kInPlace, typename T, int R, typename F>
__device__ __forceinline__ void tail_apply(const TLv<T>& L, int, const TBig<R>&, const cplx<T>* x, F&& out) {
    cplx<T> y[kBigNodes];
#pragma unroll
    for (int v = 0; v < kBigNodes; ++v) {
        const int q = thread_here() + v * kTailThreads;
        y[v] = {T(0), T(0)};
        if (q < L.N) {
            const cplx<T>* xq = x + L.li(q);
            const cplx<T>* cp = L.coef + L.gi(q);
#pragma unroll 1
            for (int dy = -R; dy <= R; ++dy)
#pragma unroll
                for (int dx = -R; dx <= R; ++dx)
                    y[v] = cfma(y[v], cp[(long long)((dy + R) * (2 * R + 1) + dx + R) * L.g.plane], xq[dy * L.lp + dx]);
        }
    }
    if constexpr (kInPlace) __syncthreads();
#pragma unroll
    for (int v = 0; v < kBigNodes; ++v) {
        const int q = thread_here() + v * kTailThreads;
        if (q < L.N) out(L.li(q), y[v]);
    }
    __syncthreads();
}

// v = sigma A x for every node, a Krylov vector of the step (sums as in held_sum_wide).
template <typename T, int R>
__device__ __forceinline__ void tail_power(const TLv<T>& L, int ln, const THeld<T, R>& h, const cplx<T>* x, cplx<T>* v) {
    cplx<double> y{0.0, 0.0};
    if (ln >= 0) y = h.template apply<true>(L, ln, x);
    if (ln >= 0 && held_part() == 0) v[ln] = cast<T>(L.sigma * y);
    __syncthreads();
}
template <typename T, int R>
__device__ __forceinline__ void tail_power(const TLv<T>& L, int, const TBig<R>&, const cplx<T>* x, cplx<T>* v) {
    tnodes(L, [&](int q) {
        const cplx<T>* xq = x + L.li(q);
        const cplx<T>* cp = L.coef + L.gi(q);
        cplx<double> y{0.0, 0.0};
#pragma unroll 1
        for (int dy = -R; dy <= R; ++dy)
#pragma unroll
            for (int dx = -R; dx <= R; ++dx)
                y = cfma(y, cast<double>(cp[(long long)((dy + R) * (2 * R + 1) + dx + R) * L.g.plane]),
                         cast<double>(xq[dy * L.lp + dx]));
        v[L.li(q)] = cast<T>(L.sigma * y);
    });
    __syncthreads();
}

// f(l) for the nodes of a level, a thread per node, l the LDS index.
template <typename H, typename T, typename F>
__device__ __forceinline__ void tail_nodes(const TLv<T>& L, F&& f) {
    if constexpr (H::kHeld) {
        const int q = thread_here();
        if (q < L.N) f(L.li(q));
    } else {
        tnodes(L, [&](int q) { f(L.li(q)); });
    }
}

// nu weighted-Jacobi sweeps (§3)
template <typename T, typename H>
__device__ __forceinline__ void tail_jacobi(const TLv<T>& L, int ln, const H& h, double inv_omega, int nu) {
    constexpr int R = H::kRadius, C = (2 * R + 1) * R + R;  // centre coefficient (c[0] of the lane that calls out)
    const T w = T(inv_omega);
    cplx<T>* u = L.u();
    const cplx<T>* f = L.f();
    for (int s = 0; s < nu; ++s)
        tail_apply<true>(L, ln, h, u, [&](int l, cplx<T> y) {
            cplx<T> d;
            if constexpr (H::kHeld) d = h.c[0];
            else d = L.coef[(long long)C * L.g.plane + L.g.at(l % L.lp - kTailGhost, l / L.lp - kTailGhost)];
            u[l] = u[l] + w * cdiv(f[l] - y, d);
        });
}

// Shared words of the reduction of a GMRES step.
template <typename T>
struct TailShared {
    GramReal<T> part[kTailWaves][kGram];
    GmWeights<T> w;
};

// The step's weights from v_0 .. v_3 (planes): each wavefront that has nodes
// sums the Gram entries over them, the first adds the wavefronts' sums and solves.
template <typename H, typename T>
__device__ __forceinline__ GmWeights<T> tail_weights(const TLv<T>& L, const cplx<T>* v0, const cplx<T>* v1,
                                                     const cplx<T>* v2, const cplx<T>* v3, TailShared<T>& sh) {
    using R = GramReal<T>;
    const int t = thread_here(), wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int wn = min((L.N + 63) >> 6, kTailWaves);
    if (wave < wn) {
        GramAcc<T> acc;
        acc.clear();
        tail_nodes<H>(L, [&](int l) {
            const cplx<T> v[4] = {v0[l], v1[l], v2[l], v3[l]};
            acc.add(v);
        });
        R s[kGram];
#pragma unroll
        for (int k = 0; k < kGram; ++k) {
            if constexpr (sizeof(T) == 8) s[k] = two_sum(acc.s[k], acc.l[k]);
            else s[k] = acc.s[k];
        }
        const R sum = wave_sum16(s);
        if ((lane & 3) == 0) sh.part[wave][gram_slot(lane)] = sum;
    }
    __syncthreads();
    if (wave == 0) {
        const R sum = sum_rows(sh.part, wn, lane);
        GmWeights<T> w;
        weights_of<T>(sum, GmBasis{L.sigma, {0.0, 0.0, 0.0}, kPivotMin<T>}, w);
        if (lane == 0) sh.w = w;
    }
    __syncthreads();
    return sh.w;
}

// One GMRES(3) smoothing step (§5.3). from_zero: u holds zeros (the level was
// just entered by restriction), so the first residual is f, read in place. res
// (may be null): a plane other than r, v_1, v_2 that receives the residual
// f - A u' of the updated iterate, by recurrence.
template <typename T, typename H>
__device__ __forceinline__ void tail_gmres(const TLv<T>& L, int ln, const H& h, TailShared<T>& sh, bool from_zero,
                                           cplx<T>* res) {
    cplx<T>* u = L.u();
    const cplx<T>* f = L.f();
    cplx<T>* v1 = L.s(1);
    cplx<T>* v2 = L.s(2);
    cplx<T>* v3 = L.s(3);
    if (!from_zero) {
        cplx<T>* r = L.s(0);
        tail_apply<false>(L, ln, h, u, [&](int l, cplx<T> y) { r[l] = f[l] - y; });
    }
    const cplx<T>* v0 = from_zero ? f : L.s(0);
    tail_power(L, ln, h, v0, v1);
    tail_power(L, ln, h, v1, v2);
    tail_power(L, ln, h, v2, v3);
    const GmWeights<T> w = tail_weights<H>(L, v0, v1, v2, v3, sh);
    tail_nodes<H>(L, [&](int l) {
        const cplx<T> a = v0[l], b = v1[l], c = v2[l], d = v3[l];
        cplx<T> x = u[l];
        if (w.k > 0) x = cfma(x, w.cu[0], a);
        if (w.k > 1) x = cfma(x, w.cu[1], b);
        if (w.k > 2) x = cfma(x, w.cu[2], c);
        u[l] = x;
        if (res) {  // read before the store: res may be the plane of v_3
            cplx<T> r = cfma(cplx<T>{T(0), T(0)}, w.cr[0], a);
            if (w.k > 0) r = cfma(r, w.cr[1], b);
            if (w.k > 1) r = cfma(r, w.cr[2], c);
            if (w.k > 2) r = cfma(r, w.cr[3], d);
            res[l] = r;
        }
    });
    __syncthreads();
}

// f_c = R w (§4 transfers, R = P^T / 4) for the fine residual in plane s(3), and
// u_c = 0; the LDS frame supplies the zero ghosts that truncate the mask at the
// boundary.
template <typename T>
__device__ __forceinline__ void tail_restrict(const TLv<T>& L, const TLv<T>& C, bool bez) {
    const cplx<T>* w = L.s(3);
    const T w0 = bez ? T(6) : T(2), w1 = bez ? T(4) : T(1), w2 = bez ? T(1) : T(0);
    const T mw[5] = {w2, w1, w0, w1, w2};
    const T scale = T(bez ? 1.0 / 256.0 : 1.0 / 16.0);
    tnodes(C, [&](int q) {
        const int J = C.row(q), pf = (2 * J + kTailGhost) * L.lp + 2 * C.col(q, J) + kTailGhost;
        cplx<T> acc{T(0), T(0)};
#pragma unroll
        for (int dy = -2; dy <= 2; ++dy) {
            cplx<T> row{T(0), T(0)};
#pragma unroll
            for (int dx = -2; dx <= 2; ++dx) {
                const cplx<T> v = w[pf + dy * L.lp + dx];
                row.re += mw[dx + 2] * v.re;
                row.im += mw[dx + 2] * v.im;
            }
            acc.re += mw[dy + 2] * row.re;
            acc.im += mw[dy + 2] * row.im;
        }
        const int lc = C.li(q);
        C.f()[lc] = scale * acc;
        C.u()[lc] = cplx<T>{T(0), T(0)};
    });
    __syncthreads();
}

// u += P e (§4 prolongation; the zero frame of the coarse plane truncates).
template <typename T>
__device__ __forceinline__ void tail_prolong(const TLv<T>& C, const TLv<T>& L, bool bez) {
    const cplx<T>* e = C.u();
    tnodes(L, [&](int q) {
        const int j = L.row(q), i = L.col(q, j);
        T wx[3], wy[3];
        const bool ox = i & 1, oy = j & 1;
        wx[0] = ox ? T(0) : (bez ? T(0.125) : T(0));
        wx[1] = ox ? T(0.5) : (bez ? T(0.75) : T(1));
        wx[2] = ox ? T(0.5) : (bez ? T(0.125) : T(0));
        wy[0] = oy ? T(0) : (bez ? T(0.125) : T(0));
        wy[1] = oy ? T(0.5) : (bez ? T(0.75) : T(1));
        wy[2] = oy ? T(0.5) : (bez ? T(0.125) : T(0));
        const int pc = ((j >> 1) - 1 + kTailGhost) * C.lp + (i >> 1) - 1 + kTailGhost;
        cplx<T> acc{T(0), T(0)};
#pragma unroll
        for (int ty = 0; ty < 3; ++ty) {
            cplx<T> row{T(0), T(0)};
#pragma unroll
            for (int tx = 0; tx < 3; ++tx) {
                const cplx<T> v = e[pc + ty * C.lp + tx];
                row.re += wx[tx] * v.re;
                row.im += wx[tx] * v.im;
            }
            acc.re += wy[ty] * row.re;
            acc.im += wy[ty] * row.im;
        }
        const int li = L.li(q);
        L.u()[li] = L.u()[li] + acc;
    });
    __syncthreads();
}

// u = A_c^{-1} f on the coarsest level with the explicit FP64 inverse
// (complex64 data is widened): a row of sixteen lanes per row of the inverse.
template <typename T>
__device__ __forceinline__ void tail_coarse(const TLv<T>& C, const cplx<double>* inv) {
    const cplx<T>* f = C.f();
    const int tid = thread_here(), part = tid & 15;
    for (int r0 = 0; r0 < C.N; r0 += kTailThreads / 16) {
        const int r = r0 + (tid >> 4);
        cplx<double> acc{0.0, 0.0};
        if (r < C.N)
            for (int p = part; p < C.N; p += 16) acc = cfma(acc, inv[(long long)r * C.N + p], cast<double>(f[C.li(p)]));
        acc = cplx<double>{acc.re + dpp_move<0x128, 0xF>(acc.re), acc.im + dpp_move<0x128, 0xF>(acc.im)};
        acc = cplx<double>{acc.re + dpp_move<0x124, 0xF>(acc.re), acc.im + dpp_move<0x124, 0xF>(acc.im)};
        acc = cplx<double>{acc.re + dpp_move<0x4e, 0xF>(acc.re), acc.im + dpp_move<0x4e, 0xF>(acc.im)};
        acc = cplx<double>{acc.re + dpp_move<0xb1, 0xF>(acc.re), acc.im + dpp_move<0xb1, 0xF>(acc.im)};
        if (r < C.N && part == 0) C.u()[C.li(r)] = cast<T>(acc);
    }
    __syncthreads();
}

// R0: stencil radius of the tail's first level, R1: of the levels below it.
template <typename T, int R0, int R1>
__global__ __launch_bounds__(kTailThreads) void k_tail(TailArgs<T> a, const int* active) {
    const int b = blockIdx.x;
    if (!rhs_active(active, b)) return;
    __shared__ TailShared<T> sh;
    cplx<T>* lds = reinterpret_cast<cplx<T>*>(hm_dyn_lds);
    const int last = a.nlev - 1;
    // zero every plane (the frames must read zero), stage the coarsest
    // inverse in LDS when it fits, then load the top level
    {
        const long long total = a.plane_bytes / (long long)sizeof(cplx<T>);
        for (long long q = threadIdx.x; q < total; q += kTailThreads) lds[q] = cplx<T>{T(0), T(0)};
        if (a.inv_off >= 0) {
            const int N = (a.lv[last].g.n + 1) * (a.lv[last].g.n + 1);
            cplx<double>* dst = reinterpret_cast<cplx<double>*>(hm_dyn_lds + a.inv_off);
            for (int q = threadIdx.x; q < N * N; q += kTailThreads) dst[q] = a.inv[q];
        }
        const TLv<T> L = tail_level(a, 0, lds);
        const long long off = (long long)b * L.g.plane;
        const bool load_u = a.top_zero == 0;  // otherwise the zeroed plane is the iterate
        cplx<T> fv[kBigNodes], uv[kBigNodes];
#pragma unroll
        for (int v = 0; v < kBigNodes; ++v) {
            const int q = thread_here() + v * kTailThreads;
            if (q < L.N) {
                fv[v] = a.f_top[off + L.gi(q)];
                if (load_u) uv[v] = a.u_top[off + L.gi(q)];
            }
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < kBigNodes; ++v) {
            const int q = thread_here() + v * kTailThreads;
            if (q < L.N) {
                L.f()[L.li(q)] = fv[v];
                if (load_u) L.u()[L.li(q)] = uv[v];
            }
        }
        __syncthreads();
    }
    const cplx<double>* inv = a.inv_off >= 0 ? reinterpret_cast<const cplx<double>*>(hm_dyn_lds + a.inv_off) : a.inv;
    const double inv_omega = 1.0 / a.omega;
    const bool bez = a.bez != 0;
    // f(level, LDS index of the lane's held node, tag of the stencil) for level q
    auto with_level = [&](int q, auto&& f) {
        const TLv<T> L = tail_level(a, q, lds);
        const int hn = held_node(), ln = hn < L.N ? L.li(hn) : -1;
        if (q == 0) {
            if (L.N > kTailThreads / 2) f(L, -1, TTag<TBig<R0>>{});
            else f(L, ln, TTag<THeld<T, R0>>{});
        } else {
            if (L.N > kTailThreads / 2) f(L, -1, TTag<TBig<R1>>{});
            else f(L, ln, TTag<THeld<T, R1>>{});
        }
    };
    // Cycle state machine: going down, the residual of the level above is
    // restricted to level q (unless it is a further visit) and q is pre-smoothed;
    // coming back up after its last coarse visit, the correction is prolongated and
    // q is post-smoothed.
    unsigned visits = 0u;  // 2 bits per level: coarse visits left
    int q = 0;
    bool up = false;
    bool fresh = a.top_zero != 0;  // level q holds u = 0 (entered by restriction, not yet smoothed)
    if (last == 0) {
        tail_coarse(tail_level(a, 0, lds), inv);
    } else {
        for (;;) {
            if (!up && q == last) {
                if (fresh) tail_restrict(tail_level(a, q - 1, lds), tail_level(a, q, lds), bez);
                tail_coarse(tail_level(a, q, lds), inv);
                q -= 1;
                up = true;
                continue;
            }
            if (up) {
                // back from one visit of level q + 1: u now holds a result
                fresh = false;
                const unsigned left = ((visits >> (2 * q)) & 3u) - 1u;
                visits = (visits & ~(3u << (2 * q))) | (left << (2 * q));
                if (left > 0) {
                    q += 1;
                    up = false;
                    continue;
                }
            }
            const int nu = up ? a.nu2 : a.nu1;
            with_level(q, [&](const TLv<T>& L, int ln, auto tag) {
                using H = typename decltype(tag)::type;
                H h;
                // FP32: arrives during the transfer (FP64 has no registers for both)
                constexpr bool kEarly = sizeof(T) == 4;
                if (kEarly) h.load(L);
                if (up) tail_prolong(tail_level(a, q + 1, lds), L, bez);
                else if (fresh && q > 0) tail_restrict(tail_level(a, q - 1, lds), L, bez);
                // going down, plane s(3) receives the residual f - A u to restrict
                if (a.smoother == 0 || nu == 0) {
                    if (!kEarly) h.load(L);
                    tail_jacobi<T, H>(L, ln, h, inv_omega, nu);
                    if (!up) {
                        cplx<T>* w = L.s(3);
                        const cplx<T>* f = L.f();
                        tail_apply<false>(L, ln, h, L.u(), [&](int l, cplx<T> y) { w[l] = f[l] - y; });
                    }
                } else {
                    for (int s = 0; s < nu; ++s) {
                        if (!kEarly || s > 0) h.load(L);
                        tail_gmres<T, H>(L, ln, h, sh, fresh && s == 0, !up && s + 1 == nu ? L.s(3) : nullptr);
                    }
                }
            });
            if (!up) {
                visits = (visits & ~(3u << (2 * q))) | (unsigned(a.gamma) << (2 * q));
                q += 1;
                fresh = true;
            } else {
                if (q == 0) break;
                q -= 1;
            }
        }
    }
    const TLv<T> L = tail_level(a, 0, lds);
    const long long off = (long long)b * L.g.plane;
    tnodes(L, [&](int k) { a.u_top[off + L.gi(k)] = L.u()[L.li(k)]; });
}

}  // namespace

// Calls f with the tail kernel for the radii of the first level and of those
// below it (Bézier hierarchies: 2 on level 1, 3 below; linear: 1).
template <typename T, typename F>
static void with_tail_kernel(int r0, F&& f) {
    if (r0 == 1) f(&k_tail<T, 1, 1>);
    else if (r0 == 2) f(&k_tail<T, 2, 3>);
    else f(&k_tail<T, 3, 3>);
}

void tail_init(int device) {
    static OncePerDevice once;
    once(device, [] {
        for (int r = 1; r <= 3; ++r) {
            auto raise = [](auto kern) {
                (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(kTailMaxLdsBytes));
            };
            with_tail_kernel<double>(r, raise);
            with_tail_kernel<float>(r, raise);
        }
    });
}

template <typename T>
void launch_tail(const LaunchCtx& ctx, const TailArgs<T>& args) {
    with_tail_kernel<T>(args.lv[0].radius, [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(ctx.nrhs), dim3(kTailThreads), size_t(args.lds_bytes), ctx.stream, args,
                           ctx.active);
    });
}
template void launch_tail<double>(const LaunchCtx&, const TailArgs<double>&);
template void launch_tail<float>(const LaunchCtx&, const TailArgs<float>&);

}  // namespace hm
