// dl_blas.hip -- Krylov vector kernels: fused BiCGStab / CGNR updates with
// their reductions, the per-right-hand-side scalar updates, and generic field
// kernels (copy/convert, norms, dots, reliable-update folding).
//
// Every launch covers a batch of segments (one per lattice); a work item is
// one (right-hand side, site block) of a segment, or one right-hand side for
// the scalar kernels.  Reductions are deterministic: each site block writes
// one partial per right-hand side, and one workgroup per right-hand side sums
// them in a fixed order.  Items whose mask flag is clear return
// at once.
#include <algorithm>

#include "dl_krylov.hpp"

namespace dl {

namespace {

constexpr int BS = 256;
constexpr int PERSIST = 8 * 32 * 16;  // grid cap of the streaming kernels (multiple of 8)

template <typename R>
__device__ __forceinline__ cx<R> ld_c(const double *p) { return {R(p[0]), R(p[1])}; }

__device__ __forceinline__ bool masked_off(const int *mask, int rhs) { return mask != nullptr && !mask[rhs]; }

// profiling: the first block of a live right-hand side counts it once
__device__ __forceinline__ void count_live(unsigned *live, int blk)
{
    if (live != nullptr && blk == 0 && threadIdx.x == 0) atomicAdd(live, 1u);
}

// ---------------------------------------------------------------- scalar kernels (one workgroup per rhs)

constexpr int SCALAR_WAVES = 4;  // at most, per right-hand side

// out[k] = sum over blocks of partials [rhs][nblk][NP] component k, in a fixed
// order; valid in thread 0.  All components of a block's partial are read
// together (they are neighbours in memory) and four blocks are in flight per
// lane, so the sum costs a few memory latencies instead of one per component
// and 64 blocks: with one wavefront per right-hand side and a component at a
// time the omega step of 24 right-hand sides at 24^3 x 48 (5184 blocks, seven
// sums) took 81 us, see scalar_threads for the wavefronts.
template <int NP>
__device__ void sum_parts(const double *parts, int rhs, int nblk, double out[NP])
{
    __shared__ double red[SCALAR_WAVES * NP];
    const double *q = parts + (int64_t)rhs * nblk * NP;
    const int bd = blockDim.x;
#pragma unroll
    for (int k = 0; k < NP; ++k) out[k] = 0;
    int b = threadIdx.x;
    for (; b + 3 * bd < nblk; b += 4 * bd) {
        double v[4][NP];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < NP; ++k) v[u][k] = q[(int64_t)(b + u * bd) * NP + k];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < NP; ++k) out[k] += v[u][k];
    }
    for (; b < nblk; b += bd)
#pragma unroll
        for (int k = 0; k < NP; ++k) out[k] += q[(int64_t)b * NP + k];
#pragma unroll
    for (int k = 0; k < NP; ++k) out[k] = wave_sum(out[k]);
    if (bd == 64) return;
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < NP; ++k) red[wid * NP + k] = out[k];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NP; ++k)
            for (int w = 1; w < (bd >> 6); ++w) out[k] += red[w * NP + k];
    __syncthreads();  // the next sum may overwrite red
}

__device__ void bicg_init(const SSeg &a, const SParams &p, int rhs)
{
    double b2;
    sum_parts<1>(a.parts, rhs, a.nblk, &b2);
    if (threadIdx.x != 0) return;
    KState s = {};
    s.rho[0] = s.alpha[0] = s.omega[0] = 1.0;
    s.b2 = b2;
    s.stop2 = p.tol2 * b2;
    s.delta2 = p.delta2;
    s.maxiter = p.maxiter;
    s.done = b2 > 0 ? 0 : 1;
    s.fresh = 1;
    a.st[rhs] = s;
    a.act[rhs] = b2 > 0 ? 3 : 0;  // 3: iterating, the iterate is still zero
    a.upd[rhs] = 0;
    a.restart[rhs] = 0;
}

// partials [.., 2]: (rhat, r)
__device__ void bicg_rho(const SSeg &a, int rhs)
{
    if (masked_off(a.mask, rhs)) return;
    double rn[2];
    sum_parts<2>(a.parts, rhs, a.nblk, rn);
    if (threadIdx.x != 0) return;
    KState s = a.st[rhs];
    bicg_rho_step(s, rn);
    if (s.nonfinite) {
        a.act[rhs] = 0;
        a.upd[rhs] = 0;
    }
    a.st[rhs] = s;
}

// partials [.., 1]: |r|^2
__device__ void bicg_check(const SSeg &a, const SParams &p, int rhs)
{
    if (!a.act[rhs]) return;
    double rr;
    sum_parts<1>(a.parts, rhs, a.nblk, &rr);
    if (threadIdx.x != 0) return;
    KState s = a.st[rhs];
    int act = 1, upd = a.upd[rhs];
    bicg_check_step(s, rr, s.delta2, s.maxiter, p.mixed, act, upd);
    s.fresh = 0;
    a.act[rhs] = act;
    a.upd[rhs] = upd;
    a.st[rhs] = s;
}

__device__ void bicg_alpha(const SSeg &a, int rhs)
{
    if (!a.act[rhs]) return;
    double rv[2];
    sum_parts<2>(a.parts, rhs, a.nblk, rv);
    if (threadIdx.x != 0) return;
    KState s = a.st[rhs];
    cdiv(s.rho, rv, s.alpha);
    if (!isfinite(s.alpha[0]) || !isfinite(s.alpha[1])) s.alpha[0] = s.alpha[1] = 0.0;
    a.st[rhs] = s;
}

// partials of the hop that made t ([.., 7]): (t, s), |t|^2, (rhat, t), (rhat, s).
// Its epilogue reads the vectors of the last dot anyway: the s update, which
// summed it before, moves three half fields instead of four.
__device__ void bicg_omega(const SSeg &a, int rhs)
{
    if (!a.act[rhs]) return;
    double d[7];
    sum_parts<7>(a.parts, rhs, a.nblk, d);
    if (threadIdx.x != 0) return;
    KState s = a.st[rhs];
    bicg_omega_step(s, d);
    a.st[rhs] = s;
}

// partials [.., 3]: |r|^2 of the FP64 residual, (rhat, r) of the replaced r.  A
// mixed-precision iterate was folded into the FP64 solution: it starts from zero.
__device__ void bicg_update(const SSeg &a, const SParams &p, int rhs)
{
    if (!a.upd[rhs]) {
        if (threadIdx.x == 0) a.restart[rhs] = 0;
        return;
    }
    double d[3];
    sum_parts<3>(a.parts, rhs, a.nblk, d);
    if (threadIdx.x != 0) return;
    KState s = a.st[rhs];
    int act = a.act[rhs] != 0, restart;
    bicg_update_step(s, d + 1, d[0], s.maxiter, act, restart);
    if (p.mixed) s.fresh = 1;
    a.act[rhs] = act && p.mixed ? 3 : act;
    a.restart[rhs] = restart;
    a.upd[rhs] = 0;
    a.st[rhs] = s;
}

__device__ void cg_init(const SSeg &a, const SParams &p, int rhs)
{
    double rr;
    sum_parts<1>(a.parts, rhs, a.nblk, &rr);
    if (threadIdx.x != 0) return;
    KState s = {};
    s.rr = rr;
    s.maxiter = p.maxiter;
    a.st[rhs] = s;
    a.act[rhs] = (rr > 0 && p.maxiter > 0) ? 1 : 0;
}

// alpha = |r|^2 / |Mhat p|^2 (= (p, Mhat^+ Mhat p)), partials [.., 1]
__device__ void cg_alpha(const SSeg &a, int rhs)
{
    if (!a.act[rhs]) return;
    if (a.act[rhs] == 2) {  // finished last iteration (its x update is done): now inactive
        if (threadIdx.x == 0) a.act[rhs] = 0;
        return;
    }
    double pq;
    sum_parts<1>(a.parts, rhs, a.nblk, &pq);
    if (threadIdx.x != 0) return;
    KState s = a.st[rhs];
    if (pq > 0) {
        s.alpha[0] = s.rr / pq;
    } else {  // exact convergence: nothing left to do
        s.alpha[0] = 0;
        a.act[rhs] = 0;
    }
    s.alpha[1] = 0;
    a.st[rhs] = s;
}

__device__ void cg_beta(const SSeg &a, int rhs)
{
    if (!a.act[rhs]) return;
    double rr;
    sum_parts<1>(a.parts, rhs, a.nblk, &rr);
    if (threadIdx.x != 0) return;
    KState s = a.st[rhs];
    s.beta[0] = s.rr > 0 ? rr / s.rr : 0;
    s.beta[1] = 0;
    s.rr = rr;
    s.iters += 1;
    // finished: 2 keeps it live for this iteration's x update (V_CG_P)
    if (s.iters >= s.maxiter || !(rr > 0)) a.act[rhs] = 2;
    a.st[rhs] = s;
}

__device__ void sum_out(const SSeg &a, int rhs)
{
    double v;
    sum_parts<1>(a.parts, rhs, a.nblk, &v);
    if (threadIdx.x == 0) a.out[rhs] = v;
}

template <int OP>
__global__ __launch_bounds__(64 * SCALAR_WAVES) void scalar_kernel(Segs<SSeg> B, SParams p)
{
    for_each_item(B, [&](const SSeg &a, int rhs) {
        if constexpr (OP == S_BICG_INIT) bicg_init(a, p, rhs);
        else if constexpr (OP == S_BICG_RHO) bicg_rho(a, rhs);
        else if constexpr (OP == S_BICG_ALPHA) bicg_alpha(a, rhs);
        else if constexpr (OP == S_BICG_OMEGA) bicg_omega(a, rhs);
        else if constexpr (OP == S_BICG_CHECK) bicg_check(a, p, rhs);
        else if constexpr (OP == S_BICG_UPDATE) bicg_update(a, p, rhs);
        else if constexpr (OP == S_CG_INIT) cg_init(a, p, rhs);
        else if constexpr (OP == S_CG_ALPHA) cg_alpha(a, rhs);
        else if constexpr (OP == S_CG_BETA) cg_beta(a, rhs);
        else sum_out(a, rhs);
    });
}

// ---------------------------------------------------------------- vector kernels

template <int NP>
__device__ __forceinline__ void write_parts(double v[NP], double *red, double *parts, int rhs, int nb, int blk)
{
    block_sum<NP>(v, red);
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NP; ++k) parts[((int64_t)rhs * nb + blk) * NP + k] = v[k];
    __syncthreads();
}

// f[0..4] by operation:
//   V_BICG_S   s = r - alpha v (in r's storage)                                     f: r, v
//   V_BICG_XRP x += alpha p + omega s; r = s - omega t; p = r + beta (p - omega v);
//              parts |r|^2                                                          f: x, r(s), p, t, v
//   V_CG_P     x += alpha p; p = r + beta p                                         f: p, r, x
//   V_ZERO     f0 = 0
//   V_NORM2    parts |f0|^2 + |f1|^2
//   V_RESTART  rhat = p = r; parts (rhat, r)                                        f: r, rhat, p
template <typename S, int OP>
__device__ __forceinline__ void vec_item(const VSeg &a, int item, double *red)
{
    using R = typename Fmt<S>::R;
    const int nb = (int)((a.Vh + BS - 1) / BS);
    const int rhs = item / nb, blk = item - rhs * nb;
    const int flag = a.mask != nullptr ? __builtin_amdgcn_readfirstlane(a.mask[rhs]) : 1;
    if (!flag) return;
    count_live(a.live, blk);
    const int64_t Vh = a.Vh;
    const int64_t cb = (int64_t)blk * BS + threadIdx.x;
    const bool valid = cb < Vh;
    if constexpr (OP == V_BICG_S) {
        if (!valid) return;
        const cx<R> alpha = ld_c<R>(a.st[rhs].alpha);
        cx<R> rv[12], vv[12];
        load_spinor<S, true>(a.f[0], Vh, rhs, cb, rv);
        load_spinor<S, true>(a.f[1], Vh, rhs, cb, vv);
#pragma unroll
        for (int e = 0; e < 12; ++e) rv[e] = rv[e] - alpha * vv[e];
        store_spinor<S, true>(a.f[0], Vh, rhs, cb, rv);
    } else if constexpr (OP == V_BICG_XRP) {
        double part[1] = {0};
        if (valid) {
            const KState &k = a.st[rhs];
            const cx<R> alpha = ld_c<R>(k.alpha), omega = ld_c<R>(k.omega), beta = ld_c<R>(k.beta);
            cx<R> xv[12], sv[12], pv[12], tv[12], vv[12];
            // An iterate that is still zero (the mask says so) is neither cleared nor
            // read.  FP64, one wavefront per SIMD, asks for it after the other four
            // fields: 24 right-hand sides at 8^3 x 16 27.1 us (34.0 asked for first,
            // 29.2 without the branch; 288 at 16^3 x 32 the same either way); FP32 is
            // 1% slower that way (12 right-hand sides at 12^3 x 24 34.6 and 33.8 us).
            constexpr bool LATE = sizeof(R) == 8;
            auto load_x = [&]() {
                if (!(flag & 2)) load_spinor<S, true>(a.f[0], Vh, rhs, cb, xv);
            };
#pragma unroll
            for (int e = 0; e < 12; ++e) xv[e] = {R(0), R(0)};
            if constexpr (!LATE) load_x();
            load_spinor<S, true>(a.f[1], Vh, rhs, cb, sv);
            load_spinor<S, true>(a.f[2], Vh, rhs, cb, pv);
            load_spinor<S, true>(a.f[3], Vh, rhs, cb, tv);
            load_spinor<S, true>(a.f[4], Vh, rhs, cb, vv);
            if constexpr (LATE) load_x();
#pragma unroll
            for (int e = 0; e < 12; ++e) {
                xv[e] = xv[e] + alpha * pv[e] + omega * sv[e];
                sv[e] = sv[e] - omega * tv[e];
                pv[e] = sv[e] + beta * (pv[e] - omega * vv[e]);
                part[0] += (double)sv[e].re * sv[e].re + (double)sv[e].im * sv[e].im;
            }
            store_spinor<S, true>(a.f[0], Vh, rhs, cb, xv);
            store_spinor<S, true>(a.f[1], Vh, rhs, cb, sv);
            store_spinor<S, true>(a.f[2], Vh, rhs, cb, pv);
        }
        write_parts<1>(part, red, a.parts, rhs, nb, blk);
    } else if constexpr (OP == V_CG_P) {
        if (!valid) return;
        const R alpha = R(a.st[rhs].alpha[0]), beta = R(a.st[rhs].beta[0]);
        cx<R> pv[12], rv[12], xv[12];
        load_spinor<S, true>(a.f[0], Vh, rhs, cb, pv);
        load_spinor<S, true>(a.f[1], Vh, rhs, cb, rv);
        load_spinor<S, true>(a.f[2], Vh, rhs, cb, xv);
#pragma unroll
        for (int e = 0; e < 12; ++e) {
            xv[e] = xv[e] + alpha * pv[e];
            pv[e] = rv[e] + beta * pv[e];
        }
        store_spinor<S, true>(a.f[2], Vh, rhs, cb, xv);
        store_spinor<S, true>(a.f[0], Vh, rhs, cb, pv);
    } else if constexpr (OP == V_ZERO) {
        if (!valid) return;
        cx<R> v[12];
#pragma unroll
        for (int e = 0; e < 12; ++e) v[e] = {R(0), R(0)};
        store_spinor<S, true>(a.f[0], Vh, rhs, cb, v);
    } else if constexpr (OP == V_NORM2) {
        double part[1] = {0};
        if (valid) {
            cx<R> v[12], w[12];
            load_spinor<S, true>(a.f[0], Vh, rhs, cb, v);
            load_spinor<S, true>(a.f[1], Vh, rhs, cb, w);
#pragma unroll
            for (int e = 0; e < 12; ++e)
                part[0] += ((double)v[e].re * v[e].re + (double)v[e].im * v[e].im) +
                           ((double)w[e].re * w[e].re + (double)w[e].im * w[e].im);
        }
        write_parts<1>(part, red, a.parts, rhs, nb, blk);
    } else if constexpr (OP == V_RESTART) {
        double part[2] = {0, 0};
        if (valid) {
            cx<R> v[12];
            load_spinor<S, true>(a.f[0], Vh, rhs, cb, v);
            store_spinor<S, true>(a.f[1], Vh, rhs, cb, v);
            store_spinor<S, true>(a.f[2], Vh, rhs, cb, v);
#pragma unroll
            for (int e = 0; e < 12; ++e) part[0] += (double)v[e].re * v[e].re + (double)v[e].im * v[e].im;
        }
        write_parts<2>(part, red, a.parts, rhs, nb, blk);
    }
}

template <typename S, int OP>
__global__ __launch_bounds__(BS) void vec_kernel(Segs<VSeg> B)
{
    __shared__ double red[3 * (BS / 64)];
    for_each_item(B, [&](const VSeg &a, int item) { vec_item<S, OP>(a, item, red); });
}

// dst (f0, precision SD) = src (f1, precision SS)
template <typename SD, typename SS>
__global__ __launch_bounds__(BS) void copy_kernel(Segs<VSeg> B)
{
    using RD = typename Fmt<SD>::R;
    using RS = typename Fmt<SS>::R;
    for_each_item(B, [&](const VSeg &a, int item) {
        const int nb = (int)((a.Vh + BS - 1) / BS);
        const int rhs = item / nb, blk = item - rhs * nb;
        if (masked_off(a.mask, rhs)) return;
        count_live(a.live, blk);
        const int64_t cb = (int64_t)blk * BS + threadIdx.x;
        if (cb >= a.Vh) return;
        cx<RS> v[12];
        cx<RD> w[12];
        load_spinor<SS>(a.f[1], a.Vh, rhs, cb, v);
#pragma unroll
        for (int e = 0; e < 12; ++e) w[e] = {RD(v[e].re), RD(v[e].im)};
        store_spinor<SD, true>(a.f[0], a.Vh, rhs, cb, w);
    });
}

// f0 (FP64) += f1 (precision S)      (reliable update of x; the next iteration takes
// f1 as zero, KState.fresh)
template <typename S>
__global__ __launch_bounds__(BS) void fold_kernel(Segs<VSeg> B)
{
    using R = typename Fmt<S>::R;
    for_each_item(B, [&](const VSeg &a, int item) {
        const int nb = (int)((a.Vh + BS - 1) / BS);
        const int rhs = item / nb, blk = item - rhs * nb;
        if (masked_off(a.mask, rhs)) return;
        count_live(a.live, blk);
        const int64_t cb = (int64_t)blk * BS + threadIdx.x;
        if (cb >= a.Vh) return;
        cx<double> xv[12];
        cx<R> lv[12];
        if (a.st[rhs].fresh) return;  // no iteration since the last time
        load_spinor<double, true>(a.f[0], a.Vh, rhs, cb, xv);
        load_spinor<S, true>(a.f[1], a.Vh, rhs, cb, lv);
#pragma unroll
        for (int e = 0; e < 12; ++e) {
            xv[e].re += (double)lv[e].re;
            xv[e].im += (double)lv[e].im;
        }
        store_spinor<double, true>(a.f[0], a.Vh, rhs, cb, xv);
    });
}

// The start of BiCGStab from the FP64 prepared source f0: r (f1) = rhat (f2) =
// p (f3) = f0 in the iteration precision, the FP64 solution f4 = 0; parts
// (rhat, r).  One pass instead of two copies of r, a conversion, a clear and a
// dot product.
template <typename S>
__global__ __launch_bounds__(BS) void start_kernel(Segs<VSeg> B)
{
    using R = typename Fmt<S>::R;
    __shared__ double red[2 * (BS / 64)];
    for_each_item(B, [&](const VSeg &a, int item) {
        const int nb = (int)((a.Vh + BS - 1) / BS);
        const int rhs = item / nb, blk = item - rhs * nb;
        count_live(a.live, blk);
        const int64_t cb = (int64_t)blk * BS + threadIdx.x;
        double part[2] = {0, 0};
        if (cb < a.Vh) {
            cx<double> bv[12];
            cx<R> v[12];
            load_spinor<double, true>(a.f[0], a.Vh, rhs, cb, bv);
#pragma unroll
            for (int e = 0; e < 12; ++e) v[e] = {R(bv[e].re), R(bv[e].im)};
            store_spinor<S>(a.f[1], a.Vh, rhs, cb, v);
            // the 16-bit formats round in the store: rhat, p and the norm are of the stored r
            if constexpr (Fmt<S>::VEC == 4) load_spinor<S>(a.f[1], a.Vh, rhs, cb, v);
            store_spinor<S, true>(a.f[2], a.Vh, rhs, cb, v);
            store_spinor<S, true>(a.f[3], a.Vh, rhs, cb, v);
#pragma unroll
            for (int e = 0; e < 12; ++e) part[0] += (double)v[e].re * v[e].re + (double)v[e].im * v[e].im;
#pragma unroll
            for (int e = 0; e < 12; ++e) bv[e] = {0.0, 0.0};
            store_spinor<double, true>(a.f[4], a.Vh, rhs, cb, bv);
        }
        write_parts<2>(part, red, a.parts, rhs, nb, blk);
    });
}

template <typename A>
Segs<A> make_segs(const std::vector<A> &v, int (*items)(const A &))
{
    Segs<A> B;
    if (v.empty() || v.size() > (size_t)MAXSEG) throw Error{DL_EINVAL, "internal: segment count out of range"};
    B.n = (int)v.size();
    B.prefix[0] = 0;
    for (int k = 0; k < B.n; ++k) {
        B.a[k] = v[k];
        B.prefix[k + 1] = B.prefix[k] + items(v[k]);
    }
    return B;
}

int vec_items(const VSeg &a) { return (int)((a.Vh + BS - 1) / BS) * a.nrhs; }
int scalar_items(const SSeg &a) { return a.nrhs; }

int grid_for(int total, int cap) { return total > cap ? cap : total; }

double field_rhs_bytes(int prec, int64_t Vh) { return (double)Vh * 12 * elem_bytes(prec) + (prec == P16 ? 4.0 * Vh : 0.0); }

double vec_bytes(int prec, const std::vector<VSeg> &segs, int nvec)
{
    double b = 0;
    for (const VSeg &a : segs) b += field_rhs_bytes(prec, a.Vh) * a.nrhs;
    return b * nvec;
}

// Profiled launches count the right-hand sides they process (masked ones
// move no bytes): per_rhs(Vh) bytes for each counted one.
template <typename F>
std::vector<VSeg> counted_segs(const std::vector<VSeg> &segs, ProfScope &ps, hipStream_t s, F per_rhs)
{
    std::vector<VSeg> v = segs;
    if (!prof_on() || capturing(s)) return v;
    for (VSeg &a : v) {
        a.live = prof_counter();
        if (a.live) ps.parts.push_back({a.live, per_rhs(a.Vh), 0.0, 1.0});
    }
    return v;
}

template <int OP>
void vec_dispatch(int prec, const Segs<VSeg> &B, int grid, hipStream_t s)
{
    switch (prec) {
    case P64: hipLaunchKernelGGL((vec_kernel<double, OP>), dim3(grid), dim3(BS), 0, s, B); break;
    case P32: hipLaunchKernelGGL((vec_kernel<float, OP>), dim3(grid), dim3(BS), 0, s, B); break;
    case P16: hipLaunchKernelGGL((vec_kernel<__half, OP>), dim3(grid), dim3(BS), 0, s, B); break;
    default: hipLaunchKernelGGL((vec_kernel<__hip_bfloat16, OP>), dim3(grid), dim3(BS), 0, s, B); break;
    }
}

template <typename SD>
void copy_from(int prec_src, const Segs<VSeg> &B, int grid, hipStream_t s)
{
    switch (prec_src) {
    case P64: hipLaunchKernelGGL((copy_kernel<SD, double>), dim3(grid), dim3(BS), 0, s, B); break;
    case P32: hipLaunchKernelGGL((copy_kernel<SD, float>), dim3(grid), dim3(BS), 0, s, B); break;
    case P16: hipLaunchKernelGGL((copy_kernel<SD, __half>), dim3(grid), dim3(BS), 0, s, B); break;
    default: hipLaunchKernelGGL((copy_kernel<SD, __hip_bfloat16>), dim3(grid), dim3(BS), 0, s, B); break;
    }
}

}  // namespace

int blas_blocks(int64_t Vh) { return (int)((Vh + BS - 1) / BS); }

// Wavefronts that sum a right-hand side's partials: one up to 512 blocks (eight
// partials a lane), four above, where the sums of one wavefront are a chain of
// memory latencies.  The truncated CGNR's two sums keep one at every size: the
// order of a sum then stays what its stored reference loops were made with.
static int scalar_threads(int op, const std::vector<SSeg> &segs)
{
    if (op == S_CG_INIT || op == S_CG_ALPHA || op == S_CG_BETA) return 64;
    int nblk = 0;
    for (const SSeg &a : segs) nblk = std::max(nblk, a.nblk);
    return nblk > 512 ? 64 * SCALAR_WAVES : 64;
}

void scalar_launch(int op, const std::vector<SSeg> &segs, const SParams &p, hipStream_t s)
{
    Segs<SSeg> B = make_segs(segs, scalar_items);
    const dim3 grid(grid_for(B.prefix[B.n], PERSIST)), bd(scalar_threads(op, segs));
    switch (op) {
    case S_BICG_INIT: hipLaunchKernelGGL(scalar_kernel<S_BICG_INIT>, grid, bd, 0, s, B, p); break;
    case S_BICG_RHO: hipLaunchKernelGGL(scalar_kernel<S_BICG_RHO>, grid, bd, 0, s, B, p); break;
    case S_BICG_ALPHA: hipLaunchKernelGGL(scalar_kernel<S_BICG_ALPHA>, grid, bd, 0, s, B, p); break;
    case S_BICG_OMEGA: hipLaunchKernelGGL(scalar_kernel<S_BICG_OMEGA>, grid, bd, 0, s, B, p); break;
    case S_BICG_CHECK: hipLaunchKernelGGL(scalar_kernel<S_BICG_CHECK>, grid, bd, 0, s, B, p); break;
    case S_BICG_UPDATE: hipLaunchKernelGGL(scalar_kernel<S_BICG_UPDATE>, grid, bd, 0, s, B, p); break;
    case S_CG_INIT: hipLaunchKernelGGL(scalar_kernel<S_CG_INIT>, grid, bd, 0, s, B, p); break;
    case S_CG_ALPHA: hipLaunchKernelGGL(scalar_kernel<S_CG_ALPHA>, grid, bd, 0, s, B, p); break;
    case S_CG_BETA: hipLaunchKernelGGL(scalar_kernel<S_CG_BETA>, grid, bd, 0, s, B, p); break;
    default: hipLaunchKernelGGL(scalar_kernel<S_SUM>, grid, bd, 0, s, B, p); break;
    }
}

void vec_launch(int op, int prec, const std::vector<VSeg> &segs, hipStream_t s)
{
    static const int nvec[] = {3, 8, 5, 1, 2, 3};
    ProfScope ps(PROF_BLAS, vec_bytes(prec, segs, nvec[op]), s);
    const std::vector<VSeg> sg =
        counted_segs(segs, ps, s, [&](int64_t Vh) { return nvec[op] * field_rhs_bytes(prec, Vh); });
    Segs<VSeg> B = make_segs(sg, vec_items);
    const int grid = grid_for(B.prefix[B.n], PERSIST);
    switch (op) {
    case V_BICG_S: vec_dispatch<V_BICG_S>(prec, B, grid, s); break;
    case V_BICG_XRP: vec_dispatch<V_BICG_XRP>(prec, B, grid, s); break;
    case V_CG_P: vec_dispatch<V_CG_P>(prec, B, grid, s); break;
    case V_ZERO: vec_dispatch<V_ZERO>(prec, B, grid, s); break;
    case V_NORM2: vec_dispatch<V_NORM2>(prec, B, grid, s); break;
    default: vec_dispatch<V_RESTART>(prec, B, grid, s); break;
    }
}

void start_launch(int prec, const std::vector<VSeg> &segs, hipStream_t s)
{
    const int n64 = 2, nlo = 3;
    ProfScope ps(PROF_BLAS, vec_bytes(P64, segs, n64) + vec_bytes(prec, segs, nlo), s);
    const std::vector<VSeg> sg = counted_segs(
        segs, ps, s, [&](int64_t Vh) { return n64 * field_rhs_bytes(P64, Vh) + nlo * field_rhs_bytes(prec, Vh); });
    Segs<VSeg> B = make_segs(sg, vec_items);
    const dim3 grid(grid_for(B.prefix[B.n], PERSIST));
    switch (prec) {
    case P64: hipLaunchKernelGGL(start_kernel<double>, grid, dim3(BS), 0, s, B); break;
    case P32: hipLaunchKernelGGL(start_kernel<float>, grid, dim3(BS), 0, s, B); break;
    case P16: hipLaunchKernelGGL(start_kernel<__half>, grid, dim3(BS), 0, s, B); break;
    default: hipLaunchKernelGGL(start_kernel<__hip_bfloat16>, grid, dim3(BS), 0, s, B); break;
    }
}

void copy_launch(int prec_dst, int prec_src, const std::vector<VSeg> &segs, hipStream_t s)
{
    ProfScope ps(PROF_BLAS, vec_bytes(prec_dst, segs, 1) + vec_bytes(prec_src, segs, 1), s);
    const std::vector<VSeg> sg = counted_segs(
        segs, ps, s, [&](int64_t Vh) { return field_rhs_bytes(prec_dst, Vh) + field_rhs_bytes(prec_src, Vh); });
    Segs<VSeg> B = make_segs(sg, vec_items);
    const int grid = grid_for(B.prefix[B.n], PERSIST);
    switch (prec_dst) {
    case P64: copy_from<double>(prec_src, B, grid, s); break;
    case P32: copy_from<float>(prec_src, B, grid, s); break;
    case P16: copy_from<__half>(prec_src, B, grid, s); break;
    default: copy_from<__hip_bfloat16>(prec_src, B, grid, s); break;
    }
}

void fold_launch(int prec, const std::vector<VSeg> &segs, hipStream_t s)
{
    ProfScope ps(PROF_BLAS, vec_bytes(P64, segs, 2) + vec_bytes(prec, segs, 1), s);
    const std::vector<VSeg> sg = counted_segs(
        segs, ps, s, [&](int64_t Vh) { return 2 * field_rhs_bytes(P64, Vh) + field_rhs_bytes(prec, Vh); });
    Segs<VSeg> B = make_segs(sg, vec_items);
    const int grid = grid_for(B.prefix[B.n], PERSIST);
    switch (prec) {
    case P64: hipLaunchKernelGGL(fold_kernel<double>, dim3(grid), dim3(BS), 0, s, B); break;
    case P32: hipLaunchKernelGGL(fold_kernel<float>, dim3(grid), dim3(BS), 0, s, B); break;
    case P16: hipLaunchKernelGGL(fold_kernel<__half>, dim3(grid), dim3(BS), 0, s, B); break;
    default: hipLaunchKernelGGL(fold_kernel<__hip_bfloat16>, dim3(grid), dim3(BS), 0, s, B); break;
    }
}

using U4v = unsigned __attribute__((ext_vector_type(4)));

// Streaming probe (measurement only): MODE 0 copies n 16-byte words from src
// to dst, MODE 1 reads them (the XOR of a thread's words reaches dst only if
// it equals a fixed value, so the loads stay live).  A workgroup takes tiles
// of STREAM_U x 256 contiguous words, thread t the words t, t + 256, ...: the
// STREAM_U non-temporal loads of a thread are in flight together and each
// instruction of a wavefront covers 1 KiB, the access of the field kernels
// (one 16-byte word per site and component plane).  Spreading a thread's
// loads over the whole buffer instead (grid stride) was slower: 4.7 against
// 5.5 TB/s for a copy.  Words after the last whole tile take a grid-stride
// tail.
constexpr int STREAM_U = 8;
constexpr int STREAM_GRID = 8192;

template <int MODE>
__global__ __launch_bounds__(256) void stream_kernel(const U4v *src, U4v *dst, int64_t n)
{
    const int64_t ntiles = n / (256 * STREAM_U);
    U4v acc = {0u, 0u, 0u, 0u};
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t base = tile * (256 * STREAM_U) + threadIdx.x;
        U4v v[STREAM_U];
#pragma unroll
        for (int u = 0; u < STREAM_U; ++u) v[u] = __builtin_nontemporal_load(src + base + u * 256);
#pragma unroll
        for (int u = 0; u < STREAM_U; ++u) {
            if constexpr (MODE == 0)
                __builtin_nontemporal_store(v[u], dst + base + u * 256);
            else
                acc ^= v[u];
        }
    }
    for (int64_t i = ntiles * (256 * STREAM_U) + (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * 256) {
        const U4v v = __builtin_nontemporal_load(src + i);
        if constexpr (MODE == 0)
            __builtin_nontemporal_store(v, dst + i);
        else
            acc ^= v;
    }
    if constexpr (MODE == 1)
        if (acc.x == 0x9e3779b9u && acc.y == 0x7f4a7c15u && acc.z == 0xbf58476du && acc.w == 0x94d049bbu)
            dst[blockIdx.x] = acc;
}

// nwords 16-byte words of zeros from p on (flat buffers that are no packed
// field, such as the link gradient)
__global__ __launch_bounds__(256) void fill_zero_kernel(U4v *p, int64_t n)
{
    const U4v z = {0u, 0u, 0u, 0u};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = z;
}

void zero_launch(void *p, int64_t nwords, hipStream_t s)
{
    if (nwords <= 0) return;
    const int grid = (int)std::min<int64_t>((nwords + 255) / 256, PERSIST);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, s, static_cast<U4v *>(p), nwords);
}

// Read mode writes at most one word per workgroup: dst needs STREAM_GRID x 16
// bytes (128 KiB).
void stream_launch(int mode, const void *src, void *dst, int64_t nwords, hipStream_t s)
{
    const int64_t want = (nwords + 256 * STREAM_U - 1) / (256 * STREAM_U);
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(want, STREAM_GRID));
    const U4v *a = static_cast<const U4v *>(src);
    U4v *b = static_cast<U4v *>(dst);
    if (mode == 0)
        hipLaunchKernelGGL(stream_kernel<0>, dim3(grid), dim3(256), 0, s, a, b, nwords);
    else
        hipLaunchKernelGGL(stream_kernel<1>, dim3(grid), dim3(256), 0, s, a, b, nwords);
}

}  // namespace dl
