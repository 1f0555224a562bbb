// dl_small.hip -- the whole BiCGStab solve of a small lattice in one kernel, a
// workgroup per right-hand side.
//
// A small lattice's solve is a chain of short launches: at 4^4 a BiCGStab
// iteration was nine of them, three to nine microseconds each and as much
// again between them, for arithmetic that takes a CU less.  Up to SMALL_VH
// sites per parity one parity of a field fits in LDS (96 KiB in FP64), which
// is all that a hop's threads share: the workgroup keeps the field a hop reads
// there, every thread the rest at its own sites, and barriers take the place
// of launches.  The recursion, its scalars, the convergence and
// reliable-update rules are those of the batched solver (bicg_* in
// dl_krylov.hpp); only the order of the sums differs.
#include <type_traits>

#include "dl_dslash.hpp"
#include "dl_krylov.hpp"

namespace dl {

namespace {

constexpr int NT = 256;  // threads of a workgroup: one wavefront per SIMD, with its registers to itself
constexpr int NW = NT / 64;
static_assert(SMALL_VH == 2 * NT, "two sites of a parity per thread at most");

// the 12 / WAYS components from `off` on of a stored spinor
template <typename S, int WAYS>
__device__ __forceinline__ void own_load(const Field &f, int Vh, int rhs, int j, int off, cx<typename Fmt<S>::R> *v)
{
    constexpr int V = Fmt<S>::VEC;
    using E = typename Fmt<S>::E;
    const E *p = reinterpret_cast<const E *>(spinor_base<S>(f, Vh, rhs));
#pragma unroll
    for (int e = 0; e < 12 / WAYS; ++e) {
        const int c = off + e;
        v[e] = Fmt<S>::ld(p, (c / V * plane_stride(Vh) + j) * V + c % V);
    }
}
template <typename S, int WAYS>
__device__ __forceinline__ void own_store(const Field &f, int Vh, int rhs, int j, int off,
                                          const cx<typename Fmt<S>::R> *v)
{
    constexpr int V = Fmt<S>::VEC;
    static_assert(V <= 2, "the 16-bit formats order their components differently");
    using E = typename Fmt<S>::E;
    E *p = reinterpret_cast<E *>(const_cast<char *>(spinor_base<S>(f, Vh, rhs)));
#pragma unroll
    for (int e = 0; e < 12 / WAYS; ++e) {
        const int c = off + e;
        Fmt<S>::st(p, (c / V * plane_stride(Vh) + j) * V + c % V, v[e]);
    }
}

// N sums over the workgroup, the same value in every thread, in a fixed order
template <int N>
__device__ __forceinline__ void all_sum(double v[N], double *red)
{
    const int wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = wave_sum(v[k]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) red[wid * N + k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        double s = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[w * N + k];
        v[k] = s;
    }
    __syncthreads();
}

// x + a z
template <typename R>
__device__ __forceinline__ cx<R> axpy(R a, cx<R> z, cx<R> x)
{
    x.re = fma(a, z.re, x.re);
    x.im = fma(a, z.im, x.im);
    return x;
}

template <typename R>
__device__ __forceinline__ cx<R> to_cx(const double a[2])
{
    return {R(a[0]), R(a[1])};
}

// a vector's entries at a thread's sites: in registers (one site per thread)
// or in its packed field
template <typename S, bool REG, int WAYS>
struct Own {
    using R = typename Fmt<S>::R;
    static constexpr int NC = 12 / WAYS;
    cx<R> v[REG ? NC : 1];
    __device__ __forceinline__ void get(const Field &f, int Vh, int rhs, int j, int off, cx<R> o[NC]) const
    {
        if constexpr (REG) {
#pragma unroll
            for (int e = 0; e < NC; ++e) o[e] = v[e];
        } else {
            own_load<S, WAYS>(f, Vh, rhs, j, off, o);
        }
    }
    __device__ __forceinline__ void set(const Field &f, int Vh, int rhs, int j, int off, bool valid, const cx<R> o[NC])
    {
        if constexpr (REG) {
#pragma unroll
            for (int e = 0; e < NC; ++e) v[e] = o[e];
        } else {
            if (valid) own_store<S, WAYS>(f, Vh, rhs, j, off, o);
        }
    }
};

}  // namespace

// S: the iteration precision (double or float).  K: sites of a parity per
// thread; with one the vectors stay in registers, with more they are in their
// packed fields, which the caches serve.  WAYS wavefronts share 64 sites, each
// taking the hops of 4 / WAYS directions and keeping 4 / WAYS spins of the
// vectors (2 on lattices of at most 128 sites per parity, which would leave
// half the SIMDs idle).
// The hop is instantiated once per precision: the two operators of an
// iteration are two turns of one loop, and so are an operator's two hops; the
// FP64 passes (prepared source, reliable update, reconstruction with the true
// residual) are one code with a mode.  Inlined at every use it was 100 KiB of
// instructions and spilled.
// What bounds it: one CU's FP64 rate and the chain of its waits (at 384 sites
// 52 us per iteration, 27 of them instructions being issued), whatever the
// threads: with 512 the same within 5%, links loaded two or three hops ahead
// no faster.  Measured on loops of 12 right-hand sides in FP64, whole calls
// against the batched kernels' (which later lost 200 us outside the solve on
// both sides): 4^4 2.00 -> 0.67 ms (0.45 now), 4^3 x 8 2.11 -> 1.03 (0.81),
// 4^2 x 6 x 8 2.18 -> 1.45 (1.22); of 288: 2.97 -> 1.15 (0.93), 4.14 -> 2.14
// (1.92), 4.86 -> 3.30 (3.20).
// Up to 512 sites it wins at any number of right-hand sides and in both
// precisions. Loops (kappa 0.145, 1e-10) of 1, 288 and 8192 right-hand sides,
// this kernel and the batched ones, ms: 128 sites FP64 0.41 / 1.21, 0.88 / 2.05,
// 13.6 / 23.8, FP32 0.42 / 1.22, 0.90 / 2.02, 14.2 / 16.7; 384 sites FP64 1.12 /
// 1.50, 2.80 / 3.87, 46.4 / 70.7, FP32 1.03 / 1.46, 2.28 / 3.17, 37.4 / 44.6; 512
// sites FP64 1.11 / 1.33, 3.18 / 4.50, 56.4 / 78.4, FP32 1.00 / 1.32, 2.44 /
// 3.55, 40.5 / 51.6.  From 648 on the batched kernels' many CUs win.
template <typename S, int NE, int K, int WAYS>
__global__ __launch_bounds__(NT) void small_bicg_kernel(SmallArgs A)
{
    using R = typename Fmt<S>::R;
    constexpr bool MIXED = !std::is_same<S, double>::value, REG = K == 1 && (WAYS == 2 || MIXED), MREG = K == 1;
    constexpr int NC = 12 / WAYS, SP = NT / WAYS;
    static_assert(WAYS == 1 || K == 1, "a wavefront that shares its sites has one per lane");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[7 * NW];
    __shared__ cx<double> swap[WAYS > 1 ? NW * (12 - NC) * 64 : 1];

    const Geom &g = A.g;
    const int Vh = g.Vh, rhs = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int way = wave % WAYS, off = NC * way, first = wave / WAYS * 64 + lane;
    // Threads past the last site mirror it.  The index is opaque: with one site per thread it never
    // changes, and the compiler would keep the addresses of every field's planes over the solve.
    auto site = [&](int k) {
        int j = min(first + k * SP, Vh - 1);
        asm volatile("" : "+v"(j));
        return j;
    };
    auto live = [&](int k) { return first + k * SP < Vh; };

    // the field a hop reads <- this thread's entries
    auto put = [&](int k, const auto *c) {
        using T = std::remove_const_t<std::remove_reference_t<decltype(c[0])>>;
        T *ex = reinterpret_cast<T *>(smem);
        if (live(k))
#pragma unroll
            for (int e = 0; e < NC; ++e) ex[(off + e) * Vh + site(k)] = c[e];
    };
    // this thread's entries of D applied to it, on parity `par`
    auto dhop = [&](auto type, const void *links, int par, int k, auto *out) {
        using T = decltype(type);
        using Q = typename Fmt<T>::R;
        const cx<Q> *ex = reinterpret_cast<const cx<Q> *>(smem);
        const int j = site(k);
        const Site s = decode(g, j, par);
        int nb[8];
        neighbours(g, j, s, nb);
        const Q bf = (g.tap && s.t + 1 == g.T) ? Q(-1) : Q(1);
        const Q bb = (g.tap && s.t == 0) ? Q(-1) : Q(1);
        cx<Q> acc[12];
#pragma unroll
        for (int e = 0; e < 12; ++e) acc[e] = {Q(0), Q(0)};
        // A wavefront's hops PER * way .. PER * way + PER - 1; the next one's link is loaded ahead, and
        // the fences keep further loads behind the arithmetic.
        constexpr int PER = 8 / WAYS;
        cx<Q> un[2][NE];  // as stored: completed where they are used, or the loads would be waited for
        auto link = [&](int d) {
            using E = typename Fmt<T>::E;
            const E *q = static_cast<const E *>(links) +
                         (int64_t)((d >> 1) * 2 + ((d & 1) ? 1 - par : par)) * NE * Vh + ((d & 1) ? nb[d] : j);
#pragma unroll
            for (int e = 0; e < NE; ++e) un[d & 1][e] = Fmt<T>::ld(q, e * (int64_t)Vh);
        };
        auto hop = [&](auto dir) {
            constexpr int D = decltype(dir)::value, MU = D >> 1, SG = (D & 1) ? +1 : -1;
            if constexpr (D % PER == 0) link(D);
            if constexpr (D % PER != PER - 1) link(D + 1);
            asm volatile("" ::: "memory");
            cx<Q> u[9], w[12];
#pragma unroll
            for (int e = 0; e < NE; ++e) u[e] = un[D & 1][e];
            if constexpr (NE == 6) {
                u[6] = conj(u[1] * u[5] - u[2] * u[4]);
                u[7] = conj(u[2] * u[3] - u[0] * u[5]);
                u[8] = conj(u[0] * u[4] - u[1] * u[3]);
            }
            if constexpr (MU < 3) {
#pragma unroll
                for (int e = 0; e < 12; ++e) w[e] = ex[e * Vh + nb[D]];
                hop_mul<Q, MU, SG, (D & 1) == 0>(u, w, acc);
            } else {
#pragma unroll
                for (int e = 0; e < 6; ++e) w[e] = ex[(6 * t_half<SG>() + e) * Vh + nb[D]];
                hop_mul_t<Q, SG, (D & 1) == 0>(u, w, Q(2) * ((D & 1) ? bb : bf), acc);
            }
            pin_acc<Q>(acc);
            asm volatile("" ::: "memory");
        };
        using std::integral_constant;
        if (way == 0 / PER) {
            hop(integral_constant<int, 0>());
            hop(integral_constant<int, 1>());
        }
        if (way == 2 / PER) {
            hop(integral_constant<int, 2>());
            hop(integral_constant<int, 3>());
        }
        if (way == 4 / PER) {
            hop(integral_constant<int, 4>());
            hop(integral_constant<int, 5>());
        }
        if (way == 6 / PER) {
            hop(integral_constant<int, 6>());
            hop(integral_constant<int, 7>());
        }
        // every wavefront's sum at the others' spins, in the order of the wavefronts
#pragma unroll
        for (int m = 1; m < WAYS; ++m)
#pragma unroll
            for (int e = 0; e < NC; ++e) {
                cx<Q> z = acc[e];
#pragma unroll
                for (int q = 1; q < WAYS; ++q)
                    if ((way + m) % WAYS == q) z = acc[q * NC + e];
                swap[(wave * (12 - NC) + (m - 1) * NC + e) * 64 + lane] = {(double)z.re, (double)z.im};
            }
        if (WAYS > 1) __syncthreads();
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            cx<Q> z = acc[e];
#pragma unroll
            for (int q = 1; q < WAYS; ++q)
                if (way == q) z = acc[q * NC + e];
            out[e] = z;
        }
#pragma unroll
        for (int m = 1; m < WAYS; ++m) {
            const int from = wave - way + (way + WAYS - m) % WAYS;
#pragma unroll
            for (int e = 0; e < NC; ++e) {
                const cx<double> z = swap[(from * (12 - NC) + (m - 1) * NC + e) * 64 + lane];
                out[e] = {out[e].re + Q(z.re), out[e].im + Q(z.im)};
            }
        }
    };
    auto norm2 = [](const auto *c) {
        double s = 0;
#pragma unroll
        for (int e = 0; e < NC; ++e) s += (double)c[e].re * c[e].re + (double)c[e].im * c[e].im;
        return s;
    };
    auto ld64 = [&](const Field &f, int k, cx<double> *c) { own_load<double, WAYS>(f, Vh, rhs, site(k), off, c); };
    auto st64 = [&](const Field &f, int k, const cx<double> *c) {
        if (live(k)) own_store<double, WAYS>(f, Vh, rhs, site(k), off, c);
    };

    enum Mode { START, UPDATE, FINISH };
    const double k2 = A.kappa * A.kappa;
    const Field &xf = MIXED ? A.xlo : A.x64;  // the iterate
    Own<S, REG, WAYS> r, rh, p, v, t;
    Own<S, MREG, WAYS> mid;
    Own<double, MREG, WAYS> mid64;
    KState st = {};
    double sum[7];
    int act = 0;
    Mode mode = START;
    for (;;) {
        // An FP64 pass: START    |b|^2, bhat = b_e + kappa D_eo b_o
        //               UPDATE   the iterate folded into the FP64 x, the residual bhat - Mhat x
        //               FINISH   x_o = b_o + kappa D_oe x_e, the full-lattice residual b - M x
#pragma unroll
        for (int m = 0; m < 7; ++m) sum[m] = 0;
#pragma clang loop unroll(disable)
        for (int k = 0; k < K; ++k) {
            cx<double> c[NC];
            if (mode == START) {
                ld64(A.be, k, c);
                if (live(k)) sum[0] += norm2(c);
                ld64(A.bo, k, c);
                if (live(k)) sum[0] += norm2(c);
            } else {
                ld64(A.x64, k, c);
                if (MIXED && mode == UPDATE) {
                    cx<R> x[NC];
                    own_load<S, WAYS>(A.xlo, Vh, rhs, site(k), off, x);
#pragma unroll
                    for (int e = 0; e < NC; ++e) {
                        c[e].re += (double)x[e].re;
                        c[e].im += (double)x[e].im;
                        x[e] = {R(0), R(0)};
                    }
                    st64(A.x64, k, c);
                    if (live(k)) own_store<S, WAYS>(A.xlo, Vh, rhs, site(k), off, x);
                }
            }
            put(k, c);
        }
        __syncthreads();
#pragma clang loop unroll(disable)
        for (int par = mode == START ? 0 : 1; par >= 0; --par) {
#pragma clang loop unroll(disable)
            for (int k = 0; k < K; ++k) {
                cx<double> c[NC], b[NC], x[NC];
                dhop(double(), A.links64, par, k, c);
                if (par == 1) {
                    if (mode == FINISH) {
                        ld64(A.bo, k, b);
                        double d = 0;
#pragma unroll
                        for (int e = 0; e < NC; ++e) {
                            x[e] = axpy(A.kappa, c[e], b[e]);
                            const cx<double> z = axpy(A.kappa, c[e], b[e] - x[e]);
                            d += z.re * z.re + z.im * z.im;
                            c[e] = x[e];
                        }
                        st64(A.xo, k, c);
                        if (live(k)) sum[0] += d;
                    }
                    mid64.set(A.mid64, Vh, rhs, site(k), off, live(k), c);
                } else if (mode == START) {
                    ld64(A.be, k, b);
                    cx<R> h[NC], z[NC];
#pragma unroll
                    for (int e = 0; e < NC; ++e) {
                        b[e] = axpy(A.kappa, c[e], b[e]);
                        h[e] = {R(b[e].re), R(b[e].im)};
                        c[e] = {0.0, 0.0};
                        z[e] = {R(0), R(0)};
                    }
                    st64(A.bhat, k, b);
                    st64(A.x64, k, c);
                    if (MIXED && live(k)) own_store<S, WAYS>(A.xlo, Vh, rhs, site(k), off, z);
                    r.set(A.r, Vh, rhs, site(k), off, live(k), h);
                    rh.set(A.rh, Vh, rhs, site(k), off, live(k), h);
                    p.set(A.p, Vh, rhs, site(k), off, live(k), h);
                    if (live(k)) sum[1] += norm2(h);
                } else if (mode == UPDATE) {
                    ld64(A.bhat, k, b);
                    ld64(A.x64, k, x);
                    cx<R> a[NC], q[NC], y[NC];
                    r.get(A.r, Vh, rhs, site(k), off, a);
                    p.get(A.p, Vh, rhs, site(k), off, q);
                    rh.get(A.rh, Vh, rhs, site(k), off, y);
                    double d[3] = {0, 0, 0};
#pragma unroll
                    for (int e = 0; e < NC; ++e) {
                        const cx<double> n64 = axpy(k2, c[e], b[e] - x[e]);
                        d[2] += n64.re * n64.re + n64.im * n64.im;
                        const cx<R> n = {R(n64.re), R(n64.im)};
                        q[e] = q[e] + (n - a[e]);
                        a[e] = n;
                        d[0] += (double)y[e].re * n.re + (double)y[e].im * n.im;
                        d[1] += (double)y[e].re * n.im - (double)y[e].im * n.re;
                    }
                    r.set(A.r, Vh, rhs, site(k), off, live(k), a);
                    p.set(A.p, Vh, rhs, site(k), off, live(k), q);
                    if (live(k))
#pragma unroll
                        for (int m = 0; m < 3; ++m) sum[m] += d[m];
                } else {
                    ld64(A.be, k, b);
                    ld64(A.x64, k, x);
                    double d = 0;
#pragma unroll
                    for (int e = 0; e < NC; ++e) {
                        const cx<double> z = axpy(A.kappa, c[e], b[e] - x[e]);
                        d += z.re * z.re + z.im * z.im;
                    }
                    if (live(k)) sum[0] += d;
                }
            }
            __syncthreads();
            if (par == 1) {
#pragma clang loop unroll(disable)
                for (int k = 0; k < K; ++k) {
                    cx<double> c[NC];
                    mid64.get(A.mid64, Vh, rhs, site(k), off, c);
                    put(k, c);
                }
                __syncthreads();
            }
        }
        all_sum<3>(sum, red);
        if (mode == FINISH) break;
        if (mode == START) {
            st.b2 = sum[0];
            st.stop2 = A.tol2 * st.b2;
            st.done = st.b2 > 0 ? 0 : 1;
            sum[0] = sum[1];
            sum[1] = 0;
            bicg_rho_step(st, sum);
            act = st.b2 > 0 && !st.nonfinite;
        } else {
            int restart = 0;
            st.due = 0;
            bicg_update_step(st, sum, sum[2], A.maxiter, act, restart);
            if (restart) {
                sum[0] = sum[1] = 0;
#pragma clang loop unroll(disable)
                for (int k = 0; k < K; ++k) {
                    cx<R> a[NC];
                    r.get(A.r, Vh, rhs, site(k), off, a);
                    rh.set(A.rh, Vh, rhs, site(k), off, live(k), a);
                    p.set(A.p, Vh, rhs, site(k), off, live(k), a);
                    if (live(k)) sum[0] += norm2(a);
                }
                all_sum<1>(sum, red);
                bicg_rho_step(st, sum);
                if (st.nonfinite) act = 0;
            }
        }
        mode = FINISH;
        while (act) {
            // turn 0: v = Mhat p, alpha = rho / (rhat, v), s = r - alpha v (in r)
            // turn 1: t = Mhat s with (t, s), |t|^2, (rhat, t), (rhat, s), then omega, rho, beta
#pragma clang loop unroll(disable)
            for (int turn = 0; turn < 2; ++turn) {
#pragma unroll
                for (int m = 0; m < 7; ++m) sum[m] = 0;
#pragma clang loop unroll(disable)
                for (int k = 0; k < K; ++k) {
                    cx<R> c[NC];
                    if (turn == 0)
                        p.get(A.p, Vh, rhs, site(k), off, c);
                    else
                        r.get(A.r, Vh, rhs, site(k), off, c);
                    put(k, c);
                }
                __syncthreads();
#pragma clang loop unroll(disable)
                for (int par = 1; par >= 0; --par) {
#pragma clang loop unroll(disable)
                    for (int k = 0; k < K; ++k) {
                        cx<R> c[NC];
                        dhop(S(), A.links, par, k, c);
                        if (par == 1) {
                            mid.set(A.mid, Vh, rhs, site(k), off, live(k), c);
                            continue;
                        }
                        cx<R> x[NC], y[NC];
                        if (turn == 0)
                            p.get(A.p, Vh, rhs, site(k), off, x);
                        else
                            r.get(A.r, Vh, rhs, site(k), off, x);
                        rh.get(A.rh, Vh, rhs, site(k), off, y);
                        double d[7] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                        for (int e = 0; e < NC; ++e) {
                            c[e] = axpy(R(-k2), c[e], x[e]);
                            d[0] += (double)c[e].re * x[e].re + (double)c[e].im * x[e].im;
                            d[1] += (double)c[e].re * x[e].im - (double)c[e].im * x[e].re;
                            d[2] += (double)c[e].re * c[e].re + (double)c[e].im * c[e].im;
                            d[3] += (double)y[e].re * c[e].re + (double)y[e].im * c[e].im;
                            d[4] += (double)y[e].re * c[e].im - (double)y[e].im * c[e].re;
                            d[5] += (double)y[e].re * x[e].re + (double)y[e].im * x[e].im;
                            d[6] += (double)y[e].re * x[e].im - (double)y[e].im * x[e].re;
                        }
                        if (turn == 0)
                            v.set(A.v, Vh, rhs, site(k), off, live(k), c);
                        else
                            t.set(A.t, Vh, rhs, site(k), off, live(k), c);
                        if (live(k))
#pragma unroll
                            for (int m = 0; m < 7; ++m) sum[m] += d[m];
                    }
                    __syncthreads();
                    if (par == 1) {
#pragma clang loop unroll(disable)
                        for (int k = 0; k < K; ++k) {
                            cx<R> c[NC];
                            mid.get(A.mid, Vh, rhs, site(k), off, c);
                            put(k, c);
                        }
                        __syncthreads();
                    }
                }
                all_sum<7>(sum, red);
                if (turn == 1) {
                    bicg_omega_step(st, sum);
                    break;
                }
                cdiv(st.rho, sum + 3, st.alpha);
                if (!isfinite(st.alpha[0]) || !isfinite(st.alpha[1])) st.alpha[0] = st.alpha[1] = 0.0;
                const cx<R> alpha = to_cx<R>(st.alpha);
#pragma clang loop unroll(disable)
                for (int k = 0; k < K; ++k) {
                    cx<R> a[NC], b[NC];
                    r.get(A.r, Vh, rhs, site(k), off, a);
                    v.get(A.v, Vh, rhs, site(k), off, b);
#pragma unroll
                    for (int e = 0; e < NC; ++e) a[e] = a[e] - alpha * b[e];
                    r.set(A.r, Vh, rhs, site(k), off, live(k), a);
                }
            }
            // x += alpha p + omega s, r = s - omega t, p = r + beta (p - omega v), |r|^2
            const cx<R> alpha = to_cx<R>(st.alpha), omega = to_cx<R>(st.omega), beta = to_cx<R>(st.beta);
            sum[0] = 0;
#pragma clang loop unroll(disable)
            for (int k = 0; k < K; ++k) {
                cx<R> x[NC], s[NC], q[NC], w[NC], u[NC];
                own_load<S, WAYS>(xf, Vh, rhs, site(k), off, x);
                r.get(A.r, Vh, rhs, site(k), off, s);
                p.get(A.p, Vh, rhs, site(k), off, q);
                t.get(A.t, Vh, rhs, site(k), off, w);
                v.get(A.v, Vh, rhs, site(k), off, u);
#pragma unroll
                for (int e = 0; e < NC; ++e) {
                    x[e] = x[e] + alpha * q[e] + omega * s[e];
                    s[e] = s[e] - omega * w[e];
                    q[e] = s[e] + beta * (q[e] - omega * u[e]);
                }
                if (live(k)) {
                    own_store<S, WAYS>(xf, Vh, rhs, site(k), off, x);
                    sum[0] += norm2(s);
                }
                r.set(A.r, Vh, rhs, site(k), off, live(k), s);
                p.set(A.p, Vh, rhs, site(k), off, live(k), q);
            }
            all_sum<1>(sum, red);
            int upd = 0;
            bicg_check_step(st, sum[0], A.delta2, A.maxiter, MIXED, act, upd);
            if (st.nonfinite) break;
            // A reliable update waits for the next multiple of `poll` iterations, as the batched
            // solver's does; a claimed convergence (or the iteration cap, or a breakdown) does not.
            st.due |= upd;
            if (!act || (st.due && st.iters % A.poll == 0)) {
                mode = UPDATE;
                break;
            }
        }
    }
    if (threadIdx.x == 0) {
        A.st[rhs] = st;
        A.res2[rhs] = sum[0];
    }
}

// the variant for a lattice
template <typename S, int NE>
static void small_go(const SmallArgs &A, int nrhs, hipStream_t s)
{
    auto go = [&](auto kernel, int most) {  // most: sites per parity that the variant takes
        DL_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   12 * most * 16));
        hipLaunchKernelGGL(kernel, dim3(nrhs), dim3(NT), (size_t)12 * A.g.Vh * 16, s, A);
    };
    if (A.g.Vh <= NT / 2)
        go(small_bicg_kernel<S, NE, 1, 2>, NT / 2);
    else if (A.g.Vh <= NT)
        go(small_bicg_kernel<S, NE, 1, 1>, NT);
    else
        go(small_bicg_kernel<S, NE, 2, 1>, 2 * NT);
}

void k_small_bicg(int prec, int recon, const SmallArgs &A, int nrhs, hipStream_t s)
{
    if (prec == P64) {
        if (recon == 12)
            small_go<double, 6>(A, nrhs, s);
        else
            small_go<double, 9>(A, nrhs, s);
    } else {
        if (recon == 12)
            small_go<float, 6>(A, nrhs, s);
        else
            small_go<float, 9>(A, nrhs, s);
    }
}

}  // namespace dl
