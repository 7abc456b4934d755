// Level kernels of the multigrid cycle: operator apply, residual, weighted
// Jacobi, transfers, norms, FP32 refinement, adjoint gradient.
#include <cmath>

#include "hm_level.hpp"

namespace hm {
namespace {

// ---------------------------------------------------------------- operator
template <typename Op, typename T, int BY>
__global__ __launch_bounds__(kBX * BY) void k_apply(Op op, Vec<T> x, Vec<T> y, const int* active, int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* xb = x.rhs(b);
    cplx<T>* yb = y.rhs(b);
    for_nodes_applied<Op, T>(op, rpt, [xb](long long q) { return xb[q]; },
                             [&](int, int, long long p, cplx<T>, cplx<T> ax) {
                                 yb[p] = ax;
                             });
}

// y = A_s x on level 0 with x the complex64 plane xs widened to FP64, which is
// written to x as well (the outer FGMRES keeps the FP32 cycle's result as its
// FP64 vector z_j and applies the operator to it: one pass instead of two).
template <int BY>
__global__ __launch_bounds__(kBX * BY) void k_apply_widened(FineOp<double> op, Vec<float> xs, Vec<double> x,
                                                            Vec<double> y, const int* active, int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<float>* sb = xs.rhs(b);
    cplx<double>* xb = x.rhs(b);
    cplx<double>* yb = y.rhs(b);
    for_nodes_applied_pre<FineOp<double>, double>(
        op, rpt, [sb](long long q) { return sb[q]; }, [](cplx<float> v) { return cast<double>(v); },
        [](long long) { return NoVals{}; },
        [&](int, int, long long p, NoVals, cplx<double> xv, cplx<double> ax) {
            xb[p] = xv;
            yb[p] = ax;
        });
}

template <typename Op, typename T, int BY>
__global__ __launch_bounds__(kBX * BY) void k_residual(Op op, Vec<T> x, Vec<T> f, Vec<T> r, const int* active,
                                                       int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* xb = x.rhs(b);
    const cplx<T>* fb = f.rhs(b);
    cplx<T>* rb = r.rhs(b);
    for_nodes_applied_pre<Op, T>(op, rpt, [xb](long long q) { return xb[q]; }, Ident{},
                                 [fb](long long q) { return fb[q]; },
                                 [&](int, int, long long p, cplx<T> fp, cplx<T>, cplx<T> ax) {
                                     rb[p] = fp - ax;
                                 });
}

// Weighted Jacobi of §3: y = x + (omega diag(A))^{-1} (f - A x).
template <typename Op, typename T, int BY>
__global__ __launch_bounds__(kBX * BY) void k_jacobi(Op op, Vec<T> x, Vec<T> f, Vec<T> y, T inv_omega,
                                                     const int* active, int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* xb = x.rhs(b);
    const cplx<T>* fb = f.rhs(b);
    cplx<T>* yb = y.rhs(b);
    for_nodes_applied_pre<Op, T>(op, rpt, [xb](long long q) { return xb[q]; }, Ident{},
                                 [fb](long long q) { return fb[q]; },
                                 [&](int i, int j, long long p, cplx<T> fp, cplx<T> xp, cplx<T> ax) {
                                 const cplx<T> r = fp - ax;
                                 yb[p] = xp + inv_omega * cdiv(r, op.diag(i, j, p));
                             });
}

// Two weighted-Jacobi sweeps in one pass on level 0 (temporal blocking of the
// smoother of §3): x is staged for the tile plus a halo of 2, the first sweep
// runs on the tile plus a halo of 1 (nodes off the grid hold zero, the ghosts
// the second sweep reads) into a second LDS stage, the second sweep on the
// tile. Per node the arithmetic of k_jacobi (the general form of the
// five-point operator everywhere); f and k^2 of the tile are read by both
// sweeps, the second time from cache, and the loads of each sweep are
// gathered in batches.
struct Jacobi2Stage {
    static constexpr int TA = kBX + 4;  // stage A (x): tile plus 2
    static constexpr int TB = kBX + 2;  // stage B (first sweep): tile plus 1
    __host__ __device__ static size_t values(int rows) { return size_t(TA) * (rows + 4) + size_t(TB) * (rows + 2); }
};

template <typename T, int BY>
__global__ __launch_bounds__(kBX * BY) void k_jacobi2(FineOp<T> op, Vec<T> x, Vec<T> f, Vec<T> y, T inv_omega,
                                                      const int* active, int rpt) {
    using JS = Jacobi2Stage;
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* xb = x.rhs(b);
    const cplx<T>* fb = f.rhs(b);
    cplx<T>* yb = y.rhs(b);
    const Grid& g = op.g;
    const BlockXY bt = block_xy();
    const int rows = BY * rpt;
    const int c0 = bt.x * kBX, r0 = bt.y * rows;
    cplx<T>* sa = reinterpret_cast<cplx<T>*>(hm_dyn_lds);
    cplx<T>* sb = sa + JS::TA * (rows + 4);
    constexpr int NB = FillBatch<T>::value;
    if (r0 - 2 <= g.n) {  // padding tiles of batch grids stage nothing
        // stage A: x on the tile plus 2 (zero off the grid)
        cplx<T> v[NB];
        bool ok[NB];
        for_strided_batched<NB>(
            JS::TA * (rows + 4),
            [&](int u, int q) {
                const int i = c0 - 2 + q % JS::TA, j = r0 - 2 + q / JS::TA;
                ok[u] = i >= 0 && i <= g.n && j >= 0 && j <= g.n;
                v[u] = xb[g.at(min(max(i, 0), g.n), min(max(j, 0), g.n))];
            },
            [&](int u, int q) { sa[q] = ok[u] ? v[u] : cplx<T>{T(0), T(0)}; });
        __syncthreads();
        // first sweep on the tile plus 1
        cplx<T> fv[NB];
        T kv[NB];
        for_strided_batched<NB>(
            JS::TB * (rows + 2),
            [&](int u, int q) {
                const int i = c0 - 1 + q % JS::TB, j = r0 - 1 + q / JS::TB;
                ok[u] = i >= 0 && i <= g.n && j >= 0 && j <= g.n;
                const long long p = g.at(min(max(i, 0), g.n), min(max(j, 0), g.n));
                fv[u] = fb[p];
                kv[u] = op.k2[p];
            },
            [&](int u, int q) {
                const int i = c0 - 1 + q % JS::TB, j = r0 - 1 + q / JS::TB;
                cplx<T> out{T(0), T(0)};
                if (ok[u]) {
                    const int la = (j - r0 + 2) * JS::TA + (i - c0 + 2);
                    const cplx<T> r = fv[u] - op.apply5k(i, j, kv[u], sa[la], sa[la - 1], sa[la + 1],
                                                          sa[la - JS::TA], sa[la + JS::TA]);
                    out = sa[la] + inv_omega * cdiv(r, op.diag_k(i, j, kv[u]));
                }
                sb[q] = out;
            });
    }
    __syncthreads();
    // second sweep on the tile
    cplx<T> fv[NB];
    T kv[NB];
    for_nodes_batched<NB>(
        g, rpt,
        [&](int u, long long p) {
            fv[u] = fb[p];
            kv[u] = op.k2[p];
        },
        [&](int u, int i, int j, long long p) {
            const int lb = (j - r0 + 1) * JS::TB + (i - c0 + 1);
            const cplx<T> r = fv[u] - op.apply5k(i, j, kv[u], sb[lb], sb[lb - 1], sb[lb + 1], sb[lb - JS::TB],
                                                  sb[lb + JS::TB]);
            yb[p] = sb[lb] + inv_omega * cdiv(r, op.diag_k(i, j, kv[u]));
        });
}

// ---------------------------------------------------------------- transfers
// Restriction R = P^T / 4 of the §4 prolongation: the 2D row is the outer
// product of [1 4 6 4 1]/16 (Bézier) or [1 2 1]/4 (linear) centred on the
// fine node (2I, 2J); fine ghosts are zero, which truncates at the boundary.
// The coarse iterate that the next cycle starts from (zero) is written in the
// same pass when `uc` is given.
template <typename T, bool kBez, int BY>
__global__ __launch_bounds__(kBX * BY) void k_restrict(Grid gf, Grid gc, Vec<T> r, Vec<T> fc, Vec<T> uc,
                                                       const int* active, int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* rb = r.rhs(b);
    cplx<T>* fb = fc.rhs(b);
    cplx<T>* ub = uc.p ? uc.rhs(b) : nullptr;
    for_nodes(gc, rpt, [&](int I, int J, long long pc) {
        if (ub) ub[pc] = cplx<T>{T(0), T(0)};
        const long long pf = gf.at(2 * I, 2 * J);
        cplx<T> acc{T(0), T(0)};
        if constexpr (kBez) {
            constexpr T w[5] = {T(1), T(4), T(6), T(4), T(1)};
#pragma unroll
            for (int dy = -2; dy <= 2; ++dy) {
                cplx<T> row{T(0), T(0)};
#pragma unroll
                for (int dx = -2; dx <= 2; ++dx) {
                    const cplx<T> v = rb[pf + (long long)dy * gf.pitch + dx];
                    row.re += w[dx + 2] * v.re;
                    row.im += w[dx + 2] * v.im;
                }
                acc.re += w[dy + 2] * row.re;
                acc.im += w[dy + 2] * row.im;
            }
            fb[pc] = T(1.0 / 256.0) * acc;
        } else {
            constexpr T w[3] = {T(1), T(2), T(1)};
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy) {
                cplx<T> row{T(0), T(0)};
#pragma unroll
                for (int dx = -1; dx <= 1; ++dx) {
                    const cplx<T> v = rb[pf + (long long)dy * gf.pitch + dx];
                    row.re += w[dx + 1] * v.re;
                    row.im += w[dx + 1] * v.im;
                }
                acc.re += w[dy + 1] * row.re;
                acc.im += w[dy + 1] * row.im;
            }
            fb[pc] = T(1.0 / 16.0) * acc;
        }
    });
}

// The coarse values a block of fine nodes (columns [c0, c0 + 64), rows
// [r0, r0 + rows), c0 and r0 even) reads: coarse columns c0/2 - 1 ..
// c0/2 + 32 and rows r0/2 - 1 .. (r0 + rows - 1)/2 + 1, staged in LDS.
constexpr int kProlongTW = kBX / 2 + 2;
__host__ __device__ inline int prolong_rows(int rows) { return rows / 2 + 3; }

template <typename T, bool kBez, int BY>
__global__ __launch_bounds__(kBX * BY) void k_prolong_add(Grid gc, Grid gf, Vec<T> e, Vec<T> u, const int* active,
                                                          int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* eb = e.rhs(b);
    cplx<T>* ub = u.rhs(b);
    cplx<T>* lds = reinterpret_cast<cplx<T>*>(hm_dyn_lds);
    const BlockXY bt = block_xy();
    const int rows = BY * rpt;
    const int C0 = bt.x * (kBX / 2) - 1, R0 = bt.y * (rows / 2) - 1;  // coarse origin of the LDS tile
    const int ne = kProlongTW * prolong_rows(rows);
    // coarse ghosts (index -1 and nc + 1) hold zero; indices beyond them read
    // a clamped node and store zero
    constexpr int kEBatch = 4;
    cplx<T> ev[kEBatch];
    bool ok[kEBatch];
    for_strided_batched<kEBatch>(
        ne,
        [&](int v, int q) {
            const int I = C0 + q % kProlongTW, J = R0 + q / kProlongTW;
            const int Ic = min(I, gc.n + 1), Jc = min(J, gc.n + 1);
            ok[v] = I == Ic && J == Jc;
            ev[v] = eb[gc.at(Ic, Jc)];
        },
        [&](int v, int q) { lds[q] = ok[v] ? ev[v] : cplx<T>{T(0), T(0)}; });
    __syncthreads();
    constexpr int NB = 8;
    cplx<T> uo[NB];
    for_nodes_batched<NB>(
        gf, rpt, [&](int v, long long pf) { uo[v] = ub[pf]; },
        [&](int v, int i, int j, long long pf) {
            T wx[3], wy[3];
            taps<T>(i, kBez, wx);
            taps<T>(j, kBez, wy);
            const int base = ((j >> 1) - 1 - R0) * kProlongTW + (i >> 1) - 1 - C0;
            cplx<T> acc{T(0), T(0)};
#pragma unroll
            for (int ty = 0; ty < 3; ++ty) {
                cplx<T> row{T(0), T(0)};
#pragma unroll
                for (int tx = 0; tx < 3; ++tx) {
                    const cplx<T> x = lds[base + ty * kProlongTW + tx];
                    row.re += wx[tx] * x.re;
                    row.im += wx[tx] * x.im;
                }
                acc.re += wy[ty] * row.re;
                acc.im += wy[ty] * row.im;
            }
            ub[pf] = uo[v] + acc;
        });
}

// ---------------------------------------------------------------- norms
template <typename Op, typename T, int BY>
__global__ __launch_bounds__(kBX * BY) void k_resnorm(Op op, Vec<T> x, Vec<T> f, Vec<T> r, double* pout,
                                                      const int* active, int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* xb = x.rhs(b);
    const cplx<T>* fb = f.rhs(b);
    cplx<T>* rb = r.p ? r.rhs(b) : nullptr;
    double acc[1] = {0.0};
    for_nodes_applied_pre<Op, T>(op, rpt, [xb](long long q) { return xb[q]; }, Ident{},
                                 [fb](long long q) { return fb[q]; },
                                 [&](int, int, long long p, cplx<T> fp, cplx<T>, cplx<T> ax) {
                                     const cplx<T> d = fp - ax;
                                     if (rb) rb[p] = d;
                                     acc[0] += dnorm2(d);
                                 });
    block_partials<1>(acc, pout + b * kPartStride);
}

template <typename T, int BY>
__global__ __launch_bounds__(kBX * BY) void k_norm(Grid g, Vec<T> f, double* pout, const int* active, int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<T>* fb = f.rhs(b);
    double acc[1] = {0.0};
    for_nodes(g, rpt, [&](int, int, long long p) { acc[0] += dnorm2(fb[p]); });
    block_partials<1>(acc, pout + b * kPartStride);
}

// One block per right-hand side: sum the partials of a norm kernel into
// norms[b].f2 (which = 0) or norms[b].r2 (which = 1), and take the stop test
// of a solve cycle on the latter when st.ring is set.
__global__ __launch_bounds__(kThreads) void k_sum_norms(const double* pin, int nblk_in, RhsNorms* norms, int which,
                                                        const int* active, StopTest st) {
    const int b = blockIdx.x;
    const bool act = rhs_active(active, b);
    double t[1];
    reduce_partials<1>(pin + b * kPartStride, nblk_in, t);
    if (act && thread_linear() == 0) {
        if (which == 0) {
            norms[b].f2 = t[0];
        } else {
            norms[b].r2 = t[0];
            if (st.ring) {
                const double f2 = norms[b].f2;
                const double r = sqrt(t[0] / f2);
                const double* lim = st.limits + 2 * b;
                const int stop = (!isfinite(r) || r > lim[1]) ? 2 : (r <= lim[0] ? 1 : 0);
                const int c = st.count[b] + 1;
                st.ring[((c - 1) % kReportRing) * st.stride + b] = RhsReport{f2, t[0], stop, c};
                st.count[b] = c;
                if (stop) st.active[b] = 0;
            }
        }
    }
}

// ---------------------------------------------------------------- refinement
// r32 = f - A_s x (complex64), partial sums of ||f - A_s x||^2 to pout.
template <int BY>
__global__ __launch_bounds__(kBX * BY) void k_refine_residual(FineOp<double> op, Vec<double> x, Vec<double> f,
                                                              Vec<float> r32, double* pout, const int* active,
                                                              int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<double>* xb = x.rhs(b);
    const cplx<double>* fb = f.rhs(b);
    cplx<float>* rb = r32.rhs(b);
    double acc[1] = {0.0};
    for_nodes_applied_pre<FineOp<double>, double>(op, rpt, [xb](long long q) { return xb[q]; }, Ident{},
                                                  [fb](long long q) { return fb[q]; },
                                                  [&](int, int, long long p, cplx<double> fp, cplx<double>,
                                                      cplx<double> ax) {
                                                  const cplx<double> r = fp - ax;
                                                  rb[p] = cast<float>(r);
                                                  acc[0] += dnorm2(r);
                                              });
    block_partials<1>(acc, pout + b * kPartStride);
}

template <int BY>
__global__ __launch_bounds__(kBX * BY) void k_correct_residual(FineOp<double> op, Vec<double> x_in, Vec<float> e,
                                                               Vec<double> x_out, Vec<double> f, Vec<float> r32,
                                                               double* pout, const int* active, int rpt) {
    const int b = blockIdx.z;
    if (!rhs_active(active, b)) return;
    const cplx<double>* xb = x_in.rhs(b);
    const cplx<float>* eb = e.rhs(b);
    cplx<double>* ob = x_out.rhs(b);
    const cplx<double>* fb = f.rhs(b);
    cplx<float>* rb = r32.rhs(b);
    double acc[1] = {0.0};
    struct XE {
        cplx<double> x;
        cplx<float> e;
    };
    auto xload = [xb, eb](long long q) { return XE{xb[q], eb[q]}; };
    auto xmake = [](const XE& v) { return v.x + cast<double>(v.e); };
    for_nodes_applied_pre<FineOp<double>, double>(op, rpt, xload, xmake, [fb](long long q) { return fb[q]; },
                                                  [&](int, int, long long p, cplx<double> fp, cplx<double> xp,
                                                      cplx<double> ax) {
                                                  ob[p] = xp;
                                                  const cplx<double> r = fp - ax;
                                                  rb[p] = cast<float>(r);
                                                  acc[0] += dnorm2(r);
                                              });
    block_partials<1>(acc, pout + b * kPartStride);
}

// ---------------------------------------------------------------- layout
template <typename T, typename S, int BY>
__global__ __launch_bounds__(kBX * BY) void k_copy_in(Grid g, const cplx<S>* src, Vec<T> dst, int scale_w,
                                                      int conj_, int rpt) {
    const int b = blockIdx.z;
    const long long m = g.n + 1;
    const cplx<S>* sb = src + b * m * m;
    cplx<T>* db = dst.rhs(b);
    for_nodes(g, rpt, [&](int i, int j, long long p) {
        cplx<T> v = cast<T>(sb[(long long)j * m + i]);
        if (scale_w) v = (line_w<T>(i, g.n) * line_w<T>(j, g.n)) * v;
        if (conj_) v.im = -v.im;
        db[p] = v;
    });
}

template <typename T, typename S, int BY>
__global__ __launch_bounds__(kBX * BY) void k_copy_out(Grid g, Vec<T> src, cplx<S>* dst, int scale_w, int conj_,
                                                       int rpt) {
    const int b = blockIdx.z;
    const long long m = g.n + 1;
    const cplx<T>* sb = src.rhs(b);
    cplx<S>* db = dst + b * m * m;
    for_nodes(g, rpt, [&](int i, int j, long long p) {
        cplx<T> v = sb[p];
        if (scale_w) v = (line_w<T>(i, g.n) * line_w<T>(j, g.n)) * v;
        if (conj_) v.im = -v.im;
        db[(long long)j * m + i] = cast<S>(v);
    });
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_zero(cplx<T>* p, long long count) {
    for (long long q = blockIdx.x * (long long)kThreads + threadIdx.x; q < count; q += (long long)gridDim.x * kThreads)
        p[q] = cplx<T>{T(0), T(0)};
}

__global__ __launch_bounds__(kThreads) void k_fill_words(unsigned* p, long long words, unsigned value) {
    for (long long q = blockIdx.x * (long long)kThreads + threadIdx.x; q < words; q += (long long)gridDim.x * kThreads)
        p[q] = value;
}

// ---------------------------------------------------------------- gradient
// dL/dk^2_p = sum_b Re[ mu_b,p W_p (1 + i s_p / (h k_p)) u_b,p ], mu = conj(lambda).
__global__ __launch_bounds__(kThreads) void k_grad_k2(Grid g, double h, const double* k2, Vec<double> u,
                                                      Vec<double> mu, double* out, int nrhs, int rpt) {
    const long long m = g.n + 1;
    for_nodes(g, rpt, [&](int i, int j, long long p) {
        const int n = g.n;
        const double W = line_w<double>(i, n) * line_w<double>(j, n);
        const int s = (i == 0 || i == n) + (j == 0 || j == n);
        // imaginary part of 1 + i s/(h k); zero where k = 0 (as 1/(h k) -> 0
        // is taken there; setup rejects k = 0 on the boundary anyway)
        const double kk = k2[p];
        const double bi = (s && kk > 0.0) ? double(s) / (h * sqrt(kk)) : 0.0;
        double acc = 0.0;
        for (int b = 0; b < nrhs; ++b) {
            const cplx<double> t = mu.rhs(b)[p] * u.rhs(b)[p];
            acc += W * (t.re - bi * t.im);
        }
        out[(long long)j * m + i] = acc;
    });
}

}  // namespace

// ======================================================================= launchers
template <typename T>
void launch_apply(const LaunchCtx& ctx, const LevelOp<T>& lop, Vec<T> x, Vec<T> y) {
    with_op(lop, [&](auto op) {
        using Op = decltype(op);
        const Geom q = geom_op<Op, T>(lop.g, ctx);
        HM_LAUNCH_OP(q, (k_apply<Op, T, BY>), op, x, y, HM_ACTIVE, q.rpt);
    });
}

void launch_apply_widened(const LaunchCtx& ctx, const LevelOp<double>& lop, Vec<float> xs, Vec<double> x,
                          Vec<double> y) {
    using Op = FineOp<double>;
    using T = double;
    const Op op{lop.g, lop.k2, 1.0 / (lop.h * lop.h), 2.0 / lop.h};
    const Geom q = geom_op<Op, T>(lop.g, ctx);
    HM_LAUNCH_OP(q, (k_apply_widened<BY>), op, xs, x, y, HM_ACTIVE, q.rpt);
}

template <typename T>
void launch_residual(const LaunchCtx& ctx, const LevelOp<T>& lop, Vec<T> x, Vec<T> f, Vec<T> r) {
    with_op(lop, [&](auto op) {
        using Op = decltype(op);
        const Geom q = geom_op<Op, T>(lop.g, ctx);
        HM_LAUNCH_OP(q, (k_residual<Op, T, BY>), op, x, f, r, HM_ACTIVE, q.rpt);
    });
}

template <typename T>
void launch_jacobi(const LaunchCtx& ctx, const LevelOp<T>& lop, Vec<T> x, Vec<T> f, Vec<T> y, double inv_omega) {
    with_op(lop, [&](auto op) {
        using Op = decltype(op);
        const Geom q = geom_op<Op, T>(lop.g, ctx);
        HM_LAUNCH_OP(q, (k_jacobi<Op, T, BY>), op, x, f, y, T(inv_omega), HM_ACTIVE, q.rpt);
    });
}

template <typename T>
bool launch_jacobi2(const LaunchCtx& ctx, const LevelOp<T>& lop, Vec<T> x, Vec<T> f, Vec<T> y, double inv_omega) {
    bool done = false;
    with_op(lop, [&](auto op) {
        using Op = decltype(op);
        if constexpr (std::is_same<Op, FineOp<T>>::value) {
            Geom q = geom(lop.g, Op::kHeavy, ctx);
            // rows per thread lowered until both LDS stages fit the tile bound
            auto bytes = [&](int rpt) { return Jacobi2Stage::values(q.by * rpt) * sizeof(cplx<T>); };
            while (q.rpt > 1 && bytes(q.rpt) > kMaxTileBytes) --q.rpt;
            q.grid = level_grid(lop.g, q.rpt, ctx.nrhs, q.by, ctx.nrhs_cap > 1);
            if (bytes(q.rpt) <= kMaxTileBytes) {
                with_by(q.by, [&](auto byc) {
                    constexpr int BY = decltype(byc)::value;
                    hipLaunchKernelGGL((k_jacobi2<T, BY>), q.grid, q.block, bytes(q.rpt), ctx.stream, op, x, f, y,
                                       T(inv_omega), HM_ACTIVE, q.rpt);
                });
                done = true;
            }
        }
    });
    return done;
}

template <typename T>
void launch_restrict(const LaunchCtx& ctx, Grid fine, Grid coarse, int transfer, Vec<T> r, Vec<T> fc, Vec<T> uc) {
    const Geom q = geom(coarse, false, ctx);
    if (transfer == 0) HM_LAUNCH(q, (k_restrict<T, true, BY>), fine, coarse, r, fc, uc, HM_ACTIVE, q.rpt);
    else HM_LAUNCH(q, (k_restrict<T, false, BY>), fine, coarse, r, fc, uc, HM_ACTIVE, q.rpt);
}

template <typename T>
void launch_prolong_add(const LaunchCtx& ctx, Grid coarse, Grid fine, int transfer, Vec<T> e, Vec<T> u) {
    Geom q = geom(fine, false, ctx);
    // the coarse tile is dynamic shared memory: rows per thread lowered until
    // it fits the same bound as the operator tiles
    auto bytes = [&](int rpt) { return size_t(kProlongTW) * prolong_rows(q.by * rpt) * sizeof(cplx<T>); };
    if (bytes(q.rpt) > kMaxTileBytes) {
        while (q.rpt > 1 && bytes(q.rpt) > kMaxTileBytes) --q.rpt;
        q.grid = level_grid(fine, q.rpt, ctx.nrhs, q.by, ctx.nrhs_cap > 1);
        q.nblk = int(q.grid.x * q.grid.y);
    }
    const size_t shm = bytes(q.rpt);
    with_by(q.by, [&](auto byc) {
        constexpr int BY = decltype(byc)::value;
        if (transfer == 0)
            hipLaunchKernelGGL((k_prolong_add<T, true, BY>), q.grid, q.block, shm, ctx.stream, coarse, fine, e, u,
                               HM_ACTIVE, q.rpt);
        else
            hipLaunchKernelGGL((k_prolong_add<T, false, BY>), q.grid, q.block, shm, ctx.stream, coarse, fine, e, u,
                               HM_ACTIVE, q.rpt);
    });
}

double gm_sigma(double h, int level) {
    const double hl = std::ldexp(h, level);
    return std::ldexp(1.0, 7 - int(std::lround(std::log2(8.0 / (hl * hl)))));
}

void launch_sum_norms(const LaunchCtx& ctx, int nb, RhsNorms* norms, int which, int reg = 0) {
    // 64 x 4 threads: the block reduction indexes wavefronts by threadIdx.y
    hipLaunchKernelGGL(k_sum_norms, dim3(ctx.nrhs), dim3(kBX, kBY), 0, ctx.stream, region(ctx, reg), nb, norms,
                       which, HM_ACTIVE, which == 1 ? ctx.stop : StopTest{});
}

template <typename T>
void launch_resnorm(const LaunchCtx& ctx, const LevelOp<T>& lop, Vec<T> x, Vec<T> f, RhsNorms* norms, Vec<T> r) {
    int nb = 0;
    with_op(lop, [&](auto op) {
        using Op = decltype(op);
        const Geom q = geom_op<Op, T>(lop.g, ctx);
        nb = q.nblk;
        HM_LAUNCH_OP(q, (k_resnorm<Op, T, BY>), op, x, f, r, region(ctx, 0), HM_ACTIVE, q.rpt);
    });
    launch_sum_norms(ctx, nb, norms, 1);
}

template <typename T>
void launch_norm(const LaunchCtx& ctx, Grid g, Vec<T> f, RhsNorms* norms) {
    const Geom q = geom(g, false, ctx);
    HM_LAUNCH(q, (k_norm<T, BY>), g, f, region(ctx, 0), HM_ACTIVE, q.rpt);
    launch_sum_norms(ctx, q.nblk, norms, 0);
}

// The residual norms use reduction region 1 (region 0 holds level 0's Gram sums).
void launch_refine_residual(const LaunchCtx& ctx, const LevelOp<double>& lop, Vec<double> x, Vec<double> f,
                            Vec<float> r32, RhsNorms* norms) {
    using Op = FineOp<double>;
    using T = double;
    const Geom q = geom_op<Op, T>(lop.g, ctx);
    FineOp<double> op{lop.g, lop.k2, 1.0 / (lop.h * lop.h), 2.0 / lop.h};
    HM_LAUNCH_OP(q, (k_refine_residual<BY>), op, x, f, r32, region(ctx, 1), HM_ACTIVE, q.rpt);
    launch_sum_norms(ctx, q.nblk, norms, 1, 1);
}

void launch_correct_residual(const LaunchCtx& ctx, const LevelOp<double>& lop, Vec<double> x_in, Vec<float> e,
                             Vec<double> x_out, Vec<double> f, Vec<float> r32, RhsNorms* norms) {
    using Op = FineOp<double>;
    using T = double;
    const Geom q = geom_op<Op, T>(lop.g, ctx);
    FineOp<double> op{lop.g, lop.k2, 1.0 / (lop.h * lop.h), 2.0 / lop.h};
    HM_LAUNCH_OP(q, (k_correct_residual<BY>), op, x_in, e, x_out, f, r32, region(ctx, 1), HM_ACTIVE, q.rpt);
    launch_sum_norms(ctx, q.nblk, norms, 1, 1);
}

template <typename T>
void launch_copy_in(const LaunchCtx& ctx, Grid g, const void* src, bool src_is_f32, Vec<T> dst, bool scale_w,
                    bool conj) {
    const Geom q = geom(g, false, ctx);
    if (src_is_f32)
        HM_LAUNCH(q, (k_copy_in<T, float, BY>), g, static_cast<const cplx<float>*>(src), dst, int(scale_w),
                  int(conj), q.rpt);
    else
        HM_LAUNCH(q, (k_copy_in<T, double, BY>), g, static_cast<const cplx<double>*>(src), dst, int(scale_w),
                  int(conj), q.rpt);
}

template <typename T>
void launch_copy_out(const LaunchCtx& ctx, Grid g, Vec<T> src, void* dst, bool dst_is_f32, bool scale_w, bool conj) {
    const Geom q = geom(g, false, ctx);
    if (dst_is_f32)
        HM_LAUNCH(q, (k_copy_out<T, float, BY>), g, src, static_cast<cplx<float>*>(dst), int(scale_w), int(conj),
                  q.rpt);
    else
        HM_LAUNCH(q, (k_copy_out<T, double, BY>), g, src, static_cast<cplx<double>*>(dst), int(scale_w), int(conj),
                  q.rpt);
}

template <typename T>
void launch_zero(hipStream_t s, cplx<T>* p, long long count) {
    if (count <= 0) return;
    long long blocks = (count + kThreads - 1) / kThreads;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL((k_zero<T>), dim3((unsigned)blocks), dim3(kThreads), 0, s, p, count);
}

void launch_fill_words(hipStream_t s, void* p, long long bytes, unsigned value) {
    const long long words = bytes / 4;
    if (words <= 0) return;
    long long blocks = (words + kThreads - 1) / kThreads;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_words, dim3((unsigned)blocks), dim3(kThreads), 0, s, static_cast<unsigned*>(p), words,
                       value);
}

void launch_grad_k2(const LaunchCtx& ctx, Grid g, double h, const double* k2, Vec<double> u, Vec<double> mu,
                    double* grad_k2_dense) {
    const int rpt = level_rpt(g, kBY, ctx.block_cap);
    hipLaunchKernelGGL(k_grad_k2, level_grid(g, rpt, 1, kBY), dim3(kBX, kBY), 0, ctx.stream, g, h, k2, u, mu,
                       grad_k2_dense, ctx.nrhs, rpt);
}

#define HM_INST(T)                                                                                              \
    template void launch_apply<T>(const LaunchCtx&, const LevelOp<T>&, Vec<T>, Vec<T>);                         \
    template void launch_residual<T>(const LaunchCtx&, const LevelOp<T>&, Vec<T>, Vec<T>, Vec<T>);              \
    template void launch_jacobi<T>(const LaunchCtx&, const LevelOp<T>&, Vec<T>, Vec<T>, Vec<T>, double);        \
    template bool launch_jacobi2<T>(const LaunchCtx&, const LevelOp<T>&, Vec<T>, Vec<T>, Vec<T>, double);       \
    template void launch_restrict<T>(const LaunchCtx&, Grid, Grid, int, Vec<T>, Vec<T>, Vec<T>);                \
    template void launch_prolong_add<T>(const LaunchCtx&, Grid, Grid, int, Vec<T>, Vec<T>);                     \
    template void launch_resnorm<T>(const LaunchCtx&, const LevelOp<T>&, Vec<T>, Vec<T>, RhsNorms*, Vec<T>);    \
    template void launch_norm<T>(const LaunchCtx&, Grid, Vec<T>, RhsNorms*);                                    \
    template void launch_copy_in<T>(const LaunchCtx&, Grid, const void*, bool, Vec<T>, bool, bool);             \
    template void launch_copy_out<T>(const LaunchCtx&, Grid, Vec<T>, void*, bool, bool, bool);                  \
    template void launch_zero<T>(hipStream_t, cplx<T>*, long long);

HM_INST(double)
HM_INST(float)

}  // namespace hm

