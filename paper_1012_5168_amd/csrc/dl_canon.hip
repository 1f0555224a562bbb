// dl_canon.hip -- kernels on canonical fields (complex128 [nrhs][V][4][3],
// chiral spin basis, lexicographic sites): the conversion to and from packed
// parity fields, and the FP64 operators D, D^+, M, M^+ applied to canonical
// fields directly.
//
// A canonical spinor is 192 contiguous bytes, so one lane per site loading its
// own site touches 64 cache lines per instruction (a sixteen-byte load from
// 64 places 192 bytes apart) and the texture unit, not memory, sets the pace.
// Here a wavefront owns 64 consecutive sites and moves their 12 KiB in the
// order of memory, 1 KiB per instruction, through a tile in LDS from which
// (or into which) each lane then takes its own site.  Rows of the tile are 13
// sixteen-byte words long: the lanes' rows then start in different banks.
// Both parities are converted by one kernel (each canonical line read once:
// with a kernel per parity and a lane per site, 96 FP64 fields at 16^3 x 32
// took 1157 us to pack and 1172 us to unpack, 4.2 TB/s).
#include <algorithm>

#include "dl_dslash.hpp"

namespace dl {

namespace {

constexpr int TS = 64;          // sites of a tile: one wavefront
constexpr int ROW = 13;         // sixteen-byte words of a tile row: 12 components and one of padding
constexpr int TW = TS * ROW;    // sixteen-byte words of a tile

using D2 = double __attribute__((ext_vector_type(2)));

// Word q = 64 k + lane (k = 0..11) of 64 consecutive sites is component q % 12
// of site q / 12.  192 words are 16 whole sites, so k + 3 has the component of
// k and the site 16 further on: three (site, component) pairs per lane.
struct Words {
    int site[3], comp[3];
    __device__ __forceinline__ explicit Words(int lane)
    {
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int q = m * 64 + lane;
            site[m] = q / 12;
            comp[m] = q - 12 * site[m];
        }
    }
    __device__ __forceinline__ int s(int k) const { return site[k % 3] + 16 * (k / 3); }
    __device__ __forceinline__ int c(int k) const { return comp[k % 3]; }
};

// Orders the tile's writes by some lanes before its reads by others: the LDS
// operations of one wavefront execute in order, so only the compiler must not
// move them across.
__device__ __forceinline__ void tile_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ Site lex_site(const Geom &g, int i)
{
    Site s;
    int r = i / g.X;
    s.x = i - r * g.X;
    const int r2 = r / g.Y;
    s.y = r - r2 * g.Y;
    s.t = r2 / g.Z;
    s.z = r2 - s.t * g.Z;
    return s;
}

constexpr int PW = 4;  // wavefronts per workgroup of the conversions

// canonical -> packed parity fields (odd.d == nullptr: the even one only)
template <typename S>
__global__ __launch_bounds__(TS *PW) void pack_kernel(Field even, Field odd, const D2 *canon, Geom g, int V)
{
    using R = typename Fmt<S>::R;
    __shared__ D2 tiles[PW * TW];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, rhs = blockIdx.y;
    const int base = (blockIdx.x * PW + w) * TS;
    if (base >= V) return;  // uniform across the wavefront; nothing below synchronises the workgroup
    D2 *tile = tiles + w * TW;
    const Words q(lane);
    const D2 *src = canon + ((int64_t)rhs * V + base) * 12;
    const int left = V - base;
    D2 st[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) st[k] = src[min(q.s(k), left - 1) * 12 + q.c(k)];
#pragma unroll
    for (int k = 0; k < 12; ++k) tile[q.s(k) * ROW + q.c(k)] = st[k];
    tile_fence();
    cx<double> z[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) {
        const D2 v = tile[lane * ROW + e];
        z[e] = {v.x, v.y};
    }
    to_internal(z);
    cx<R> v[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) v[e] = {R(z[e].re), R(z[e].im)};
    const int i = base + lane;
    if (lane >= left) return;
    const Site s = lex_site(g, i);
    const bool p = ((s.x + s.y + s.z + s.t) & 1) != 0;
    if (p && odd.d == nullptr) return;
    store_spinor<S>(Field{p ? odd.d : even.d, p ? odd.nrm : even.nrm}, g.Vh, rhs, i >> 1, v);
}

// packed parity fields -> canonical (odd.d == nullptr: zeros on the odd sites)
template <typename S>
__global__ __launch_bounds__(TS *PW) void unpack_kernel(Field even, Field odd, D2 *canon, Geom g, int V)
{
    using R = typename Fmt<S>::R;
    __shared__ D2 tiles[PW * TW];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, rhs = blockIdx.y;
    const int base = (blockIdx.x * PW + w) * TS;
    if (base >= V) return;  // uniform across the wavefront; nothing below synchronises the workgroup
    D2 *tile = tiles + w * TW;
    const int left = V - base;
    const int i = base + min(lane, left - 1);
    const Site s = lex_site(g, i);
    const bool p = ((s.x + s.y + s.z + s.t) & 1) != 0;
    cx<double> z[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) z[e] = {0.0, 0.0};
    if (!p || odd.d != nullptr) {
        cx<R> v[12];
        load_spinor<S>(Field{p ? odd.d : even.d, p ? odd.nrm : even.nrm}, g.Vh, rhs, i >> 1, v);
#pragma unroll
        for (int e = 0; e < 12; ++e) z[e] = {(double)v[e].re, (double)v[e].im};
        to_canonical(z);
    }
#pragma unroll
    for (int e = 0; e < 12; ++e) tile[lane * ROW + e] = D2{z[e].re, z[e].im};
    tile_fence();
    const Words q(lane);
    D2 *dst = canon + ((int64_t)rhs * V + base) * 12;
#pragma unroll
    for (int k = 0; k < 12; ++k)
        if (q.s(k) < left) dst[k * 64 + lane] = tile[q.s(k) * ROW + q.c(k)];
}

// ---------------------------------------------------------------- operators on canonical fields

struct CanonArgs {
    const D2 *in;
    D2 *out;
    const void *links;
    Geom g;
    double a;
    int V, nrhs, nblk, nsplit;
};

// the stored part of U_mu of a site of parity par (NE complex numbers), and its
// completion to three rows
template <int NE>
__device__ __forceinline__ void load_rows(const void *links, int64_t Vh, int mu, int par, int64_t cb, cx<double> *u)
{
    const D2 *p = static_cast<const D2 *>(links) + ((int64_t)(mu * 2 + par) * NE) * Vh + cb;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const D2 v = p[e * Vh];
        u[e] = {v.x, v.y};
    }
}
template <int NE>
__device__ __forceinline__ void third_row(cx<double> u[9])
{
    if constexpr (NE == 6) {
        u[6] = conj(u[1] * u[5] - u[2] * u[4]);
        u[7] = conj(u[2] * u[3] - u[0] * u[5]);
        u[8] = conj(u[0] * u[4] - u[1] * u[3]);
    }
}

template <int MU, int SG, bool FWD>
__device__ __forceinline__ void canon_hop(const cx<double> u[9], const cx<double> psi[12], double b, cx<double> acc[12])
{
    cx<double> h[6], gg[6];
    project<double, MU, SG>(psi, h);
    if constexpr (MU == 3)
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = b * h[e];
    colour_mul<double, FWD>(u, h, gg);
    reconstruct<double, MU, SG>(acc, gg);
    pin_acc<double>(acc);
}

// out = a D in (XPAY = false) or in + a D in, D or D^+ (DAG), on canonical
// fields.  A wavefront owns 64 consecutive sites and walks right-hand sides;
// per right-hand side it brings the sites' own tile and the tiles of their
// neighbours in y, z and t (and in x where a row is no divisor of 64 sites:
// XIN false) through LDS in turn, the loads of the next PF tiles in flight
// while one computes, and writes the result back through the tile.
// KEEP: the sites' links stay with the wavefront over its right-hand sides, as
// stored: those of the x and y hops in LDS, those of the z and t hops in
// registers, which lets four wavefronts share a CU's LDS.  Without it (one
// right-hand side per wavefront) each hop's link is loaded a hop ahead, and
// the registers are held to two wavefronts per SIMD.
// It takes the place of packing, two half hops and unpacking (three times the
// field traffic).  At 16^3 x 32, M on one field: 102 -> 47 us per call; D on 96
// fields: 3448 -> 1690 us.  What bounds it there: memory.  The 128 wavefronts
// of an XCD hold two timeslices at a time and fetch 2.4 times the input (the
// neighbouring timeslices are as many again, and the wavefronts drift apart),
// 4.9 TB/s with the output.  Tried: one tile in flight instead of two 1.94 ms;
// projecting before the tile (half the LDS words, but loads of half lines, two
// fetches of each into L1) 2.5-2.8 ms.
template <int NE, bool DAG, bool XPAY, bool XIN, bool KEEP>
__global__ __launch_bounds__(TS, KEEP ? 1 : 2) void canon_op_kernel(CanonArgs A)
{
    constexpr int SF = DAG ? +1 : -1;  // forward projector 1 + SF g
    constexpr int SB = -SF;
    constexpr int CTR = XIN || (XPAY && KEEP) ? 1 : 0;  // whether the own tile is read ahead
    constexpr int FIRST = XIN ? 2 : 0;        // first hop that brings a tile of its own
    constexpr int NST = CTR + 8 - FIRST;      // tiles per right-hand side
    constexpr int PF = KEEP ? 2 : 1;          // tiles whose loads are in flight
    __shared__ D2 tile[TW];
    __shared__ int from[9][TS];  // element offset of each lane's neighbours (and, last, of its own site)
    __shared__ D2 lds_links[KEEP ? 4 * NE * TS : 1];

    const Geom &g = A.g;
    const int lane = threadIdx.x;
    // XCD x takes a contiguous eighth of the site blocks, every split of the
    // right-hand sides in turn
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int share = (A.nblk + 7) / 8;
    const int split = j / share, blk = xcd * share + (j - split * share);
    if (blk >= A.nblk || split >= A.nsplit) return;
    const int chunk = (A.nrhs + A.nsplit - 1) / A.nsplit;
    const int r0 = split * chunk, r1 = min(A.nrhs, r0 + chunk);
    if (r0 >= r1) return;
    const int base = blk * TS, left = A.V - base;
    const int i = base + min(lane, left - 1);  // lanes past the last site mirror it and store nothing
    const Site s = lex_site(g, i);
    const int p = (s.x + s.y + s.z + s.t) & 1, q = 1 - p;
    const int XY = g.X * g.Y, XYZ = XY * g.Z;
    int nb[8];
    nb[0] = s.x + 1 == g.X ? i - (g.X - 1) : i + 1;
    nb[1] = s.x == 0 ? i + (g.X - 1) : i - 1;
    nb[2] = s.y + 1 == g.Y ? i - (g.Y - 1) * g.X : i + g.X;
    nb[3] = s.y == 0 ? i + (g.Y - 1) * g.X : i - g.X;
    nb[4] = s.z + 1 == g.Z ? i - (g.Z - 1) * XY : i + XY;
    nb[5] = s.z == 0 ? i + (g.Z - 1) * XY : i - XY;
    nb[6] = s.t + 1 == g.T ? i - (g.T - 1) * XYZ : i + XYZ;
    nb[7] = s.t == 0 ? i + (g.T - 1) * XYZ : i - XYZ;
#pragma unroll
    for (int d = 0; d < 8; ++d) from[d][lane] = nb[d] * 12;
    from[8][lane] = i * 12;
    const double bf = (g.tap && s.t + 1 == g.T) ? -1.0 : 1.0;
    const double bb = (g.tap && s.t == 0) ? -1.0 : 1.0;
    const int64_t Vh = g.Vh;
    auto rows_of = [&](int d, cx<double> *u) {
        const bool fwd = (d & 1) == 0;
        load_rows<NE>(A.links, Vh, d >> 1, fwd ? p : q, (fwd ? i : nb[d]) >> 1, u);
    };
    cx<double> kept[KEEP ? 4 : 1][NE];
    if constexpr (KEEP) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            cx<double> u[NE];
            rows_of(d, u);
#pragma unroll
            for (int e = 0; e < NE; ++e) lds_links[(d * NE + e) * TS + lane] = D2{u[e].re, u[e].im};
        }
#pragma unroll
        for (int d = 4; d < 8; ++d) rows_of(d, kept[d - 4]);
    }
    const Words wd(lane);
    tile_fence();

    D2 st[PF][12];
    // tile k of right-hand side r into v: k < CTR the own tile, else the neighbours of hop FIRST + k - CTR
    auto fetch = [&](int r, int k, D2 *v) {
        const D2 *src = A.in + (int64_t)r * A.V * 12;
        const int d = k < CTR ? 8 : FIRST + k - CTR;
#pragma unroll
        for (int m = 0; m < 12; ++m) v[m] = src[from[d][wd.s(m)] + wd.c(m)];
    };
    auto commit = [&](const D2 *v) {
        tile_fence();  // earlier reads of the tile
#pragma unroll
        for (int m = 0; m < 12; ++m) tile[wd.s(m) * ROW + wd.c(m)] = v[m];
        tile_fence();
    };
    auto row = [&](int k, cx<double> v[12]) {
#pragma unroll
        for (int e = 0; e < 12; ++e) {
            const D2 t = tile[k * ROW + e];
            v[e] = {t.x, t.y};
        }
    };
    cx<double> ahead[KEEP ? 1 : NE];  // without KEEP: the next hop's link
    if constexpr (!KEEP) rows_of(0, ahead);
    auto link = [&](int d, cx<double> u[9]) {
        if constexpr (KEEP) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                if (d < 4) {
                    const D2 t = lds_links[(d * NE + e) * TS + lane];
                    u[e] = {t.x, t.y};
                } else {
                    u[e] = kept[d - 4][e];
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < NE; ++e) u[e] = ahead[e];
            if (d < 7) rows_of(d + 1, ahead);
        }
        third_row<NE>(u);
    };
    auto hop = [&](int d, const cx<double> psi[12], cx<double> acc[12]) {
        cx<double> u[9];
        link(d, u);
        switch (d) {
        case 0: canon_hop<0, SF, true>(u, psi, 1.0, acc); break;
        case 1: canon_hop<0, SB, false>(u, psi, 1.0, acc); break;
        case 2: canon_hop<1, SF, true>(u, psi, 1.0, acc); break;
        case 3: canon_hop<1, SB, false>(u, psi, 1.0, acc); break;
        case 4: canon_hop<2, SF, true>(u, psi, 1.0, acc); break;
        case 5: canon_hop<2, SB, false>(u, psi, 1.0, acc); break;
        case 6: canon_hop<3, SF, true>(u, psi, bf, acc); break;
        default: canon_hop<3, SB, false>(u, psi, bb, acc); break;
        }
    };
    // right-hand side r; its tile k is in st[(OFF + k) % PF]
    auto one = [&](int r, auto off) {
        constexpr int OFF = decltype(off)::value;
        cx<double> acc[12], psi[12];
        D2 own[XPAY ? 12 : 1];  // the sites' own words, in the order of memory (held where registers allow)
#pragma unroll
        for (int e = 0; e < 12; ++e) acc[e] = {0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NST; ++k) {
            D2 *slot = st[(OFF + k) % PF];
            if (k < CTR && XPAY && KEEP)
#pragma unroll
                for (int m = 0; m < 12; ++m) own[XPAY ? m : 0] = slot[m];
            if (k >= CTR || XIN) commit(slot);
            if (k + PF < NST)
                fetch(r, k + PF, slot);
            else if (KEEP)
                fetch(r + 1 < r1 ? r + 1 : r, k + PF - NST, slot);  // (after the last right-hand side: unused)
            if (k < CTR) {
                if constexpr (XIN) {
                    row(nb[0] - base, psi);
                    hop(0, psi, acc);
                    row(nb[1] - base, psi);
                    hop(1, psi, acc);
                }
            } else {
                row(lane, psi);
                hop(FIRST + k - CTR, psi, acc);
            }
        }
        if constexpr (XPAY && !KEEP) {
            const D2 *src = A.in + ((int64_t)r * A.V + base) * 12;
#pragma unroll
            for (int m = 0; m < 12; ++m) own[m] = src[min(wd.s(m), left - 1) * 12 + wd.c(m)];
        }
        tile_fence();
#pragma unroll
        for (int e = 0; e < 12; ++e) tile[lane * ROW + e] = D2{A.a * acc[e].re, A.a * acc[e].im};
        tile_fence();
        D2 *dst = A.out + ((int64_t)r * A.V + base) * 12;
#pragma unroll
        for (int m = 0; m < 12; ++m) {
            D2 v = tile[wd.s(m) * ROW + wd.c(m)];
            if constexpr (XPAY) v += own[m];
            if (wd.s(m) < left) __builtin_nontemporal_store(v, dst + m * 64 + lane);
        }
    };
#pragma unroll
    for (int k = 0; k < PF; ++k) fetch(r0, k, st[k]);
    if constexpr (!KEEP) {
        one(r0, std::integral_constant<int, 0>());
    } else if constexpr (NST % PF == 0) {
        for (int r = r0; r < r1; ++r) one(r, std::integral_constant<int, 0>());
    } else {
        static_assert(PF <= 2, "the walk alternates between two assignments");
        for (int r = r0; r < r1; r += 2) {
            one(r, std::integral_constant<int, 0>());
            if (r + 1 < r1) one(r + 1, std::integral_constant<int, 1>());
        }
    }
}

template <int NE, bool DAG, bool XPAY, bool XIN>
void canon_go(const CanonArgs &a, bool keep, dim3 grid, hipStream_t s)
{
    if (keep)
        hipLaunchKernelGGL((canon_op_kernel<NE, DAG, XPAY, XIN, true>), grid, dim3(TS), 0, s, a);
    else
        hipLaunchKernelGGL((canon_op_kernel<NE, DAG, XPAY, XIN, false>), grid, dim3(TS), 0, s, a);
}
template <int NE, bool DAG, bool XPAY>
void canon_go(const CanonArgs &a, bool keep, dim3 grid, hipStream_t s)
{
    if (TS % a.g.X == 0)
        canon_go<NE, DAG, XPAY, true>(a, keep, grid, s);
    else
        canon_go<NE, DAG, XPAY, false>(a, keep, grid, s);
}
template <int NE>
void canon_go(const CanonArgs &a, bool dag, bool xpay, bool keep, dim3 grid, hipStream_t s)
{
    if (dag) {
        if (xpay)
            canon_go<NE, true, true>(a, keep, grid, s);
        else
            canon_go<NE, true, false>(a, keep, grid, s);
    } else {
        if (xpay)
            canon_go<NE, false, true>(a, keep, grid, s);
        else
            canon_go<NE, false, false>(a, keep, grid, s);
    }
}

}  // namespace

#define DL_CANON_DISPATCH(prec, NAME, ...)                                                              \
    do {                                                                                                \
        switch (prec) {                                                                                 \
        case P64: hipLaunchKernelGGL(NAME<double>, __VA_ARGS__); break;                                 \
        case P32: hipLaunchKernelGGL(NAME<float>, __VA_ARGS__); break;                                  \
        case P16: hipLaunchKernelGGL(NAME<__half>, __VA_ARGS__); break;                                 \
        default: hipLaunchKernelGGL(NAME<__hip_bfloat16>, __VA_ARGS__); break;                          \
        }                                                                                               \
    } while (0)

void k_pack(int prec, Field even, Field odd, const double *canon, const Geom &g, int nrhs, hipStream_t s)
{
    const int V = 2 * g.Vh;
    dim3 grid((V + TS * PW - 1) / (TS * PW), nrhs);
    DL_CANON_DISPATCH(prec, pack_kernel, grid, dim3(TS * PW), 0, s, even, odd,
                      reinterpret_cast<const D2 *>(canon), g, V);
}

void k_unpack(int prec, Field even, Field odd, double *canon, const Geom &g, int nrhs, hipStream_t s)
{
    const int V = 2 * g.Vh;
    dim3 grid((V + TS * PW - 1) / (TS * PW), nrhs);
    DL_CANON_DISPATCH(prec, unpack_kernel, grid, dim3(TS * PW), 0, s, even, odd, reinterpret_cast<D2 *>(canon), g,
                      V);
}

// The kernel's element offsets are 32 bits and its grid is blocks x splits.
bool canon_op_fits(const Geom &g) { return 2LL * g.Vh * 12 < (1LL << 31); }

void k_canon_op(const void *links, int recon, bool dag, bool xpay, double a, const void *in, void *out, const Geom &g,
                int nrhs, hipStream_t s)
{
    CanonArgs A;
    A.in = static_cast<const D2 *>(in);
    A.out = static_cast<D2 *>(out);
    A.links = links;
    A.g = g;
    A.a = a;
    A.V = 2 * g.Vh;
    A.nrhs = nrhs;
    A.nblk = (A.V + TS - 1) / TS;
    // Each XCD holds 128 wavefronts (32 CUs, four by their LDS).  Right-hand
    // sides are split over more wavefronts only until the chip has two full
    // rounds of them: a wavefront stages its links once for all it walks.
    const int64_t want = 2048;
    A.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(nrhs, want / A.nblk));
    const int share = (A.nblk + 7) / 8;
    const dim3 grid((unsigned)(8LL * share * A.nsplit));
    const bool keep = nrhs > A.nsplit;
    const double e = 16.0, vh = g.Vh;
    ProfScope ps(PROF_DSLASH, 2 * (2 * 12 * e * vh) * nrhs + 2 * vh * 4 * (recon == 12 ? 6 : 9) * e, s,
                 (!xpay && !dag) ? PROF_DSLASH_PLAIN : -1);
    if (prof_on()) prof_config(ps.kind, ps.kind2, TuneChoice{2, A.nsplit, TS, 0});
    if (recon == 12)
        canon_go<6>(A, dag, xpay, keep, grid, s);
    else
        canon_go<9>(A, dag, xpay, keep, grid, s);
}

}  // namespace dl
