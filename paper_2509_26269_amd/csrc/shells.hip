// shells.hip -- lattice kernels for Hamiltonians with more than three
// exchange shells (the paper's Pd/Fe/Ir(111) parameter set has 35 shells,
// 360 bonds per site; Supplementary Note 4, Table S1).
//
// With hundreds of offsets per site the stencil is bound by multiply-adds, not
// by HBM: a workgroup stages a tile with the halo of its disc of bonds in LDS and
// convolves it row by row (the HVP) or adds it up shell by shell (the energies,
// which keep the smaller rounding error).  The spin Hamiltonian is the one of the
// three-shell kernels (Methods, Eq. param-hamiltonian): exchange on every
// shell, interfacial DMI on the nearest-neighbour shell, uniaxial anisotropy,
// Zeeman field.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "kernels.hpp"

namespace moto {

// Rows of the disc of the first NS shells: shell[dy + GEN_RMAX][dx + GEN_RMAX]
// (-1 off the disc and at the centre) and the extent lo..hi of each row.
struct DiscRows {
    int R;
    int lo[2 * GEN_RMAX + 1], hi[2 * GEN_RMAX + 1];
    signed char shell[2 * GEN_RMAX + 1][2 * GEN_RMAX + 1];
};

constexpr DiscRows make_disc(int ns) {
    DiscRows t{};
    for (int y = 0; y <= 2 * GEN_RMAX; ++y) {
        t.lo[y] = GEN_RMAX + 1;
        t.hi[y] = -GEN_RMAX - 1;
        for (int x = 0; x <= 2 * GEN_RMAX; ++x) t.shell[y][x] = -1;
    }
    for (int s = 0; s < ns; ++s)
        for (int o = kShellGeom.start[s]; o < kShellGeom.start[s + 1]; ++o) {
            const int dx = kShellGeom.dx[o], dy = kShellGeom.dy[o], y = dy + GEN_RMAX;
            t.shell[y][dx + GEN_RMAX] = (signed char)s;
            if (dx < t.lo[y]) t.lo[y] = dx;
            if (dx > t.hi[y]) t.hi[y] = dx;
            if (dy > t.R) t.R = dy;
            if (dx > t.R) t.R = dx;
        }
    return t;
}
template <int NS>
inline constexpr DiscRows kDisc = make_disc(NS);
// fewest shells of a plan that takes the disc of NS
template <int NS>
inline constexpr int kDiscMin = NS == 10 ? 4 : NS == 20 ? 11 : 21;

// couplings (cJ zero beyond the plan's shells) and the rows that the plan's
// bonds reach, in scalar registers
template <class T, int NS>
struct GenCoef {
    T cJ[NS];
    T cD, cK, B[3];
    int R;
};

// HX x HY output sites a workgroup, HSP consecutive ones of a row a thread
template <class T, int NS, int HX_, int HY_, int HSP_>
struct GenTile {
    static constexpr int HX = HX_, HY = HY_, HSP = HSP_;
    static constexpr int TPR = HX / HSP, NTH = TPR * HY;
    static constexpr int V = 16 / sizeof(T);  // values of an aligned 16-byte LDS read
    static constexpr int RY = kDisc<NS>.R, RX = (RY + V - 1) / V * V;
    static constexpr int LX = HX + 2 * RX, LY = HY + 2 * RY;
    // row stride: two rows' reads at 16-byte steps fall on different halves of
    // the 32 bytes between neighbouring threads
    static constexpr int LS = LX + V;
    T u[3][LY][LS];
};

// acc[q] += sum over the row's bonds of cJ[shell] u(q + dx)
template <class T, int NS, class TL, int DY>
struct DiscRow {
    static constexpr int LO = kDisc<NS>.lo[DY + GEN_RMAX], HI = kDisc<NS>.hi[DY + GEN_RMAX];
    // 16-byte aligned window from the first value needed
    static constexpr int W0 = (TL::RX + LO) / TL::V * TL::V;
    static constexpr int WN = (TL::RX + HI + TL::HSP - W0 + TL::V - 1) / TL::V * TL::V;

    static __device__ __forceinline__ void load(const T* __restrict__ row, T (&win)[WN]) {
        typedef T VT __attribute__((ext_vector_type(TL::V)));
#pragma unroll
        for (int i = 0; i < WN; i += TL::V) {
            const VT v = *reinterpret_cast<const VT*>(row + W0 + i);
#pragma unroll
            for (int e = 0; e < TL::V; ++e) win[i + e] = v[e];
        }
    }
    template <int I>
    static __device__ __forceinline__ void term(const T (&win)[WN], const GenCoef<T, NS>& k, T (&acc)[TL::HSP]) {
        constexpr int S = kDisc<NS>.shell[DY + GEN_RMAX][LO + I + GEN_RMAX];
        if constexpr (S >= 0) {
#pragma unroll
            for (int q = 0; q < TL::HSP; ++q) acc[q] += k.cJ[S] * win[TL::RX + LO + I - W0 + q];
        }
    }
    template <int... I>
    static __device__ __forceinline__ void terms(std::integer_sequence<int, I...>, const T (&win)[WN],
                                                 const GenCoef<T, NS>& k, T (&acc)[TL::HSP]) {
        (term<I>(win, k, acc), ...);
    }
    // the row's terms unless no bond of the plan lies in it (a zero coupling
    // would carry a non-finite value there)
    static __device__ __forceinline__ void row(const T (&win)[WN], const GenCoef<T, NS>& k, T (&acc)[TL::HSP]) {
        constexpr auto dxs = std::make_integer_sequence<int, HI - LO + 1>{};
        constexpr int Y = DY < 0 ? -DY : DY;
        if constexpr (Y > kDisc<kDiscMin<NS>>.R) {
            if (Y <= k.R) terms(dxs, win, k, acc);
        } else {
            terms(dxs, win, k, acc);
        }
    }
    // rows DY and on, each with the next one's window on its way
    static __device__ __forceinline__ void run(const T* __restrict__ base, const T (&win)[WN],
                                               const GenCoef<T, NS>& k, T (&acc)[TL::HSP]) {
        if constexpr (DY < TL::RY) {
            using Next = DiscRow<T, NS, TL, DY + 1>;
            T nxt[Next::WN];
            Next::load(base + (DY + 1 + TL::RY) * TL::LS, nxt);
            row(win, k, acc);
            __builtin_amdgcn_sched_barrier(0);  // two windows live
            Next::run(base, nxt, k, acc);
        } else {
            row(win, k, acc);
        }
    }
};

template <class T, int NS, class TL>
__device__ __forceinline__ void disc_rows(const T* __restrict__ base, const GenCoef<T, NS>& k, T (&acc)[TL::HSP]) {
    using First = DiscRow<T, NS, TL, -TL::RY>;
    T win[First::WN];
    First::load(base, win);
    First::run(base, win, k, acc);
}

// Field (A u) at the thread's HSP sites (lx0.., ly0), without anisotropy.
// The disc is unrolled: every bond is one multiply-add with its coupling as a
// scalar operand and its neighbour in a register, each row's window being read
// once in 16-byte pieces.  The earlier form convolved the full 25 x 23 square
// with couplings from LDS (1725 multiply-adds a site-vector instead of 1083,
// and a quarter as many LDS reads again), a workgroup taking the vectors one
// after another.  us of the HVP, before and now, 35 shells: 64 x 128x128 x 4 FP32
// 471 and 162 (115 for the multiply-adds alone at the vector rate; 186 with each
// row's window read in front of its own terms, the tile staged four sites at a
// time and stores by the field's owner), FP64 1137 and 241; one 128x128 state x 4
// FP32 212 and 20; 16x16 x 1 53 and 20.  A zero coupling of the disc still meets
// the sites of the plan's rows beyond its shells (up to 11 along the row), so a
// non-finite vector entry shows there too, as it did in the square.
template <class T, int NS, class TL>
__device__ __forceinline__ void disc_field(const TL& L, int lx0, int ly0, const GenCoef<T, NS>& k,
                                           T (&a)[TL::HSP][3]) {
#pragma unroll 1
    for (int cc = 0; cc < 3; ++cc) {
        T acc[TL::HSP];
#pragma unroll
        for (int q = 0; q < TL::HSP; ++q) acc[q] = T(0);
        disc_rows<T, NS, TL>(&L.u[cc][ly0][lx0], k, acc);
#pragma unroll
        for (int q = 0; q < TL::HSP; ++q) {
            a[q][0] = cc == 0 ? acc[q] : a[q][0];
            a[q][1] = cc == 1 ? acc[q] : a[q][1];
            a[q][2] = cc == 2 ? acc[q] : a[q][2];
        }
    }
    // nearest-neighbour DMI
    if (k.cD != T(0)) {
        constexpr int NDX[6] = {1, 0, -1, -1, 0, 1}, NDY[6] = {0, 1, 1, 0, -1, -1};
#pragma unroll
        for (int o = 0; o < 6; ++o) {
            const T hx = k.cD * (T(NDX[o]) + T(0.5) * T(NDY[o]));
            const T hy = k.cD * (T(0.86602540378443864676) * T(NDY[o]));
#pragma unroll
            for (int q = 0; q < TL::HSP; ++q) {
                const int y = ly0 + TL::RY + NDY[o], x = lx0 + TL::RX + q + NDX[o];
                const T u0 = L.u[0][y][x], u1 = L.u[1][y][x], u2 = L.u[2][y][x];
                a[q][0] += hx * u2;
                a[q][1] += hy * u2;
                a[q][2] -= hx * u0 + hy * u1;
            }
        }
    }
}

struct GenPos {
    int id, b, tx0, ty0;
};
template <class TL>
__device__ __forceinline__ GenPos gen_pos(const Geo& g, int id) {
    GenPos t;
    const int ntx = (g.Lx + TL::HX - 1) / TL::HX, nty = (g.Ly + TL::HY - 1) / TL::HY;
    t.id = id;
    t.b = id / (ntx * nty);
    const int r = id - t.b * ntx * nty;
    t.tx0 = (r % ntx) * TL::HX;
    t.ty0 = (r / ntx) * TL::HY;
    return t;
}

// Fill the staged tile: ld(site index, raw[NR]) reads, mk(raw, u[3]) makes the
// staged vector.  A thread's sites are read 10 at a time, all loads in flight
// (35 shells, 64 x 128x128 x 4 FP32, 18.6 sites a thread: 182 us with four, 169).
template <class TL, int NR, class LD, class MK>
__device__ __forceinline__ void stage_gen(TL& L, const Geo& g, const GenPos& t, LD&& ld, MK&& mk) {
    using T = std::remove_reference_t<decltype(L.u[0][0][0])>;
    constexpr int SITES = TL::LX * TL::LY, PER = (SITES + TL::NTH - 1) / TL::NTH;
    constexpr int U = PER < 10 ? PER : 10;
#pragma unroll 1
    for (int i0 = threadIdx.x; i0 < SITES; i0 += U * TL::NTH) {
        T raw[U][NR];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int i = min(i0 + q * TL::NTH, SITES - 1);
            const int ly = i / TL::LX, lx = i - ly * TL::LX;
            ld(wrap1(t.tx0 + lx - TL::RX, g.Lx) + g.Lx * wrap1(t.ty0 + ly - TL::RY, g.Ly), raw[q]);
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int i = i0 + q * TL::NTH;
            const int ly = i / TL::LX, lx = i - ly * TL::LX;
            T u[3];
            mk(raw[q], u);
            if (i < SITES) {
#pragma unroll
                for (int d = 0; d < 3; ++d) L.u[d][ly][lx] = u[d];
            }
        }
    }
}

// Field (A u) at one site of a staged tile, shell by shell: the members of a
// shell are added first, then scaled by its coupling.  The energies of both
// precisions keep this order: disc_field's running sum over up to 360 bonds has
// 2.1 times its rms error (35 shells, against 80-bit sums), in FP32 enough to
// show in an FP64 energy, and its zero couplings carry a non-finite spin beyond
// the plan's shells.  It is unrolled, so that every neighbour is an LDS read at
// an immediate offset; shells beyond the plan's are skipped.  us of the energy
// and gradient, 35 shells, with the offsets from a table, through disc_field and
// now: 64 x 128x128 FP32 158, -, 77, FP64 298, 68, 133; 512 x 16x16 FP64 102, 60,
// 39 (disc_field's 64 x 32 tiles mostly empty).
template <class T, int NS, class TL, int S, int... I>
__device__ __forceinline__ void shell_add(std::integer_sequence<int, I...>, const TL& L, int y, int x,
                                          const GenCoef<T, NS>& k, T (&a)[3]) {
    T m[3] = {T(0), T(0), T(0)};
    constexpr int O = kShellGeom.start[S];
    ((m[0] += L.u[0][y + kShellGeom.dy[O + I]][x + kShellGeom.dx[O + I]],
      m[1] += L.u[1][y + kShellGeom.dy[O + I]][x + kShellGeom.dx[O + I]],
      m[2] += L.u[2][y + kShellGeom.dy[O + I]][x + kShellGeom.dx[O + I]]),
     ...);
#pragma unroll
    for (int d = 0; d < 3; ++d) a[d] += k.cJ[S] * m[d];
    __builtin_amdgcn_sched_barrier(0);  // one shell's neighbours live at a time
}
template <class T, int NS, class TL, int... S>
__device__ __forceinline__ void shells_add(std::integer_sequence<int, S...>, const TL& L, int y, int x, int ns,
                                           const GenCoef<T, NS>& k, T (&a)[3]) {
    ((S < ns ? shell_add<T, NS, TL, S>(
                   std::make_integer_sequence<int, kShellGeom.start[S + 1] - kShellGeom.start[S]>{}, L, y, x, k, a)
             : void()),
     ...);
}
template <class T, int NS, class TL>
__device__ __forceinline__ void shell_field(const TL& L, int lx0, int ly0, int ns, const GenCoef<T, NS>& k,
                                            T (&a)[3]) {
    const int y = ly0 + TL::RY, x = lx0 + TL::RX;
    a[0] = a[1] = a[2] = T(0);
    shells_add<T, NS, TL>(std::make_integer_sequence<int, NS>{}, L, y, x, ns, k, a);
    if (k.cD != T(0)) {
#pragma unroll
        for (int o = 0; o < 6; ++o) {
            const int ddx = kShellGeom.dx[o], ddy = kShellGeom.dy[o];
            const T u0 = L.u[0][y + ddy][x + ddx], u1 = L.u[1][y + ddy][x + ddx], u2 = L.u[2][y + ddy][x + ddx];
            const T hx = k.cD * (T(ddx) + T(0.5) * T(ddy));
            const T hy = k.cD * (T(0.86602540378443864676) * T(ddy));
            a[0] += hx * u2;
            a[1] += hy * u2;
            a[2] -= hx * u0 + hy * u1;
        }
    }
}

// Output site q of a thread: consecutive lanes on consecutive sites of a row, for
// the global loads and stores.
template <class TL>
struct GenSite {
    int x, y;
    __device__ __forceinline__ GenSite(int q) {
        const int i = threadIdx.x + q * TL::NTH;
        x = i % TL::HX;
        y = i / TL::HX;
    }
};

// Staged vector and field of the thread's output sites.  disc_field gives a thread
// HSP consecutive sites of a row; they change hands through the tile (spent by
// then), since loads and stores 32 bytes apart touch eight times the cache
// lines (10 shells, 64 x 128x128 x 4 FP32: 96 -> 78 us).
template <class T, int NS, class TL>
__device__ __forceinline__ void site_fields(TL& L, const GenCoef<T, NS>& k, T (&u)[TL::HSP][3], T (&a)[TL::HSP][3]) {
    static_assert(TL::HX * TL::HY == TL::HSP * TL::NTH, "every thread has HSP output sites");
#pragma unroll
    for (int q = 0; q < TL::HSP; ++q) {
        const GenSite<TL> o(q);
#pragma unroll
        for (int d = 0; d < 3; ++d) u[q][d] = L.u[d][o.y + TL::RY][o.x + TL::RX];
    }
    const int lx0 = (threadIdx.x % TL::TPR) * TL::HSP, ly0 = threadIdx.x / TL::TPR;
    disc_field<T, NS>(L, lx0, ly0, k, a);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TL::HSP; ++q)
#pragma unroll
        for (int d = 0; d < 3; ++d) L.u[d][ly0][lx0 + q] = a[q][d];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TL::HSP; ++q) {
        const GenSite<TL> o(q);
#pragma unroll
        for (int d = 0; d < 3; ++d) a[q][d] = L.u[d][o.y][o.x];
    }
}

// Energy, gradient, c, F of the general-shell Hamiltonian, a site a thread;
// part[tile] = sum_i (1/2 m_i.(A m)_i - B.m_i).
template <class T, int NS>
using EnergyTile = GenTile<T, NS, 32, 16, 1>;
template <class T, int NS>
__global__ __launch_bounds__(512) void k_energy_grad_gen(Geo g, int ns, int tile0, GenCoef<T, NS> k,
                                                         const T* __restrict__ m,
                                                         const uint8_t* __restrict__ mask, T* __restrict__ grad,
                                                         T* __restrict__ cout, T* __restrict__ F,
                                                         double* __restrict__ part) {
    using TL = EnergyTile<T, NS>;
    static_assert(TL::NTH == 512, "a site a thread");
    __shared__ __align__(16) TL L;
    __shared__ double red[TL::NTH / 64];
    const GenPos t = gen_pos<TL>(g, tile0 + blockIdx.x);
    const size_t N = g.N;
    const T* mb = m + (size_t)t.b * 3 * N;
    stage_gen<TL, 3>(
        L, g, t,
        [&](int s, T(&r)[3]) {
#pragma unroll
            for (int d = 0; d < 3; ++d) r[d] = mb[d * N + s];
        },
        [](const T(&r)[3], T(&u)[3]) {
#pragma unroll
            for (int d = 0; d < 3; ++d) u[d] = r[d];
        });
    __syncthreads();
    const GenSite<TL> o(0);
    const int x = t.tx0 + o.x, y = t.ty0 + o.y;
    T mi[3], ai[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) mi[d] = L.u[d][o.y + TL::RY][o.x + TL::RX];
    shell_field<T, NS>(L, o.x, o.y, ns, k, ai);
    double v = 0.0;
    if (x < g.Lx && y < g.Ly) {
        const size_t s = x + (size_t)g.Lx * y, s1 = (size_t)t.b * N + s, s3 = (size_t)t.b * 3 * N + s;
        ai[2] += k.cK * mi[2];
        const T gi[3] = {ai[0] - k.B[0], ai[1] - k.B[1], ai[2] - k.B[2]};
        const T ci = mi[0] * gi[0] + mi[1] * gi[1] + mi[2] * gi[2];
        if (grad) {
#pragma unroll
            for (int d = 0; d < 3; ++d) grad[s3 + d * N] = gi[d];
        }
        if (cout) cout[s1] = ci;
        if (F) {
            const bool act = mask == nullptr || mask[s1] != 0;
#pragma unroll
            for (int d = 0; d < 3; ++d) F[s3 + d * N] = act ? -(gi[d] - ci * mi[d]) : T(0);
        }
        const double mam = (double)mi[0] * ai[0] + (double)mi[1] * ai[1] + (double)mi[2] * ai[2];
        const double bm = (double)k.B[0] * mi[0] + (double)k.B[1] * mi[1] + (double)k.B[2] * mi[2];
        v = 0.5 * mam - bm;
    }
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < TL::NTH / 64; ++w) s += red[w];
        part[t.id] = s;
    }
}

// Tangent HVP (frame or ambient layout, as the three-shell kernels): one tile
// of one vector a workgroup, a tile's vectors on one XCD (they share its spins:
// 35 shells, 64 x 128x128 x 4 FP32 167 -> 161 us, 10 shells 78 -> 70),
// W_j = M H(m) M V_j with (H v)_i = P_i (A v)_i - c_i v_i.
template <class T, bool FRAME, int NS, class TL>
__global__ __launch_bounds__(TL::NTH) void k_tangent_hvp_gen(Geo g, GenCoef<T, NS> k, const T* __restrict__ m,
                                                             const T* __restrict__ c,
                                                             const uint8_t* __restrict__ mask, int nvec,
                                                             long long vbs, const T* __restrict__ V,
                                                             T* __restrict__ W, DoneFlags done) {
    constexpr int DV = FRAME ? 2 : 3;
    __shared__ __align__(16) TL L;
    const int id = xcd_order(true), j = id % nvec;
    const GenPos t = gen_pos<TL>(g, id / nvec);
    if (done(t.b)) return;
    const size_t N = g.N;
    const T* mb = m + (size_t)t.b * 3 * N;
    const uint8_t* mk = mask ? mask + (size_t)t.b * N : nullptr;
    const T* vj = V + (size_t)t.b * vbs + (size_t)j * DV * N;
    T* wj = W + (size_t)t.b * vbs + (size_t)j * DV * N;
    constexpr int NR = FRAME ? 5 : 3;  // coordinates, then the spin of the frame
    stage_gen<TL, NR>(
        L, g, t,
        [&](int s, T(&r)[NR]) {
            const bool on = mk == nullptr || mk[s] != 0;
#pragma unroll
            for (int d = 0; d < DV; ++d) r[d] = on ? vj[d * N + s] : T(0);
            if constexpr (FRAME) {
#pragma unroll
                for (int d = 0; d < 3; ++d) r[2 + d] = mb[d * N + s];
            }
        },
        [](const T(&r)[NR], T(&u)[3]) {
            if constexpr (FRAME) {
                T f1[3], f2[3];
                onb(r[2], r[3], r[4], f1, f2);
#pragma unroll
                for (int d = 0; d < 3; ++d) u[d] = fma(r[0], f1[d], r[1] * f2[d]);
            } else {
#pragma unroll
                for (int d = 0; d < 3; ++d) u[d] = r[d];
            }
        });
    __syncthreads();
    T us[TL::HSP][3], a[TL::HSP][3];
    site_fields<T, NS>(L, k, us, a);
#pragma unroll
    for (int q = 0; q < TL::HSP; ++q) {
        const GenSite<TL> o(q);
        const int x = t.tx0 + o.x, y = t.ty0 + o.y;
        if (x >= g.Lx || y >= g.Ly) continue;
        const size_t so = x + (size_t)g.Lx * y;
        const bool on = mk == nullptr || mk[so] != 0;
        const T(&u)[3] = us[q];
        const T ci = c[(size_t)t.b * N + so];
        const T m0 = mb[so], m1 = mb[N + so], m2 = mb[2 * N + so];
        const T a0 = a[q][0], a1 = a[q][1], a2 = a[q][2] + k.cK * u[2];
        if constexpr (FRAME) {
            T e1[3], e2[3];
            onb(m0, m1, m2, e1, e2);
            const T av = e1[0] * u[0] + e1[1] * u[1] + e1[2] * u[2];
            const T bv = e2[0] * u[0] + e2[1] * u[1] + e2[2] * u[2];
            const T wa = e1[0] * a0 + e1[1] * a1 + e1[2] * a2 - ci * av;
            const T wb = e2[0] * a0 + e2[1] * a1 + e2[2] * a2 - ci * bv;
            wj[so] = on ? wa : T(0);
            wj[N + so] = on ? wb : T(0);
        } else {
            const T ma = m0 * a0 + m1 * a1 + m2 * a2;
            wj[so] = on ? a0 - ma * m0 - ci * u[0] : T(0);
            wj[N + so] = on ? a1 - ma * m1 - ci * u[1] : T(0);
            wj[2 * N + so] = on ? a2 - ma * m2 - ci * u[2] : T(0);
        }
    }
}

// --------------------------------------------------------------------------
template <class TL>
static long long gen_tiles(const Geo& g) {
    return (long long)((g.Lx + TL::HX - 1) / TL::HX) * ((g.Ly + TL::HY - 1) / TL::HY);
}

// Calls f(couplings, shells) for the precision and the smallest disc of 10, 20
// or 36 shells (5, 8 and 11 rows of halo) that holds the plan's.
template <class T, class F>
static void with_disc(const CoefD& kd, F&& f) {
    auto go = [&](auto nsc) {
        constexpr int NS = decltype(nsc)::value;
        GenCoef<T, NS> k;
        for (int s = 0; s < NS; ++s) k.cJ[s] = s < kd.gen->ns ? (T)kd.gen->cJ[s] : T(0);
        k.cD = (T)kd.cD;
        k.cK = (T)kd.cK;
        for (int d = 0; d < 3; ++d) k.B[d] = (T)kd.B[d];
        k.R = kd.gen->R;
        f(k, nsc);
    };
    if (kd.gen->ns <= 10)
        go(std::integral_constant<int, 10>{});
    else if (kd.gen->ns <= 20)
        go(std::integral_constant<int, 20>{});
    else
        go(std::integral_constant<int, GEN_MAX_SHELLS>{});
}

// Calls f(tile): 64 x 32 sites (2.1 staged sites an output for 36 shells)
// where `copies` lattices of them fill the chip twice, 32 x 16 (4.2) where
// they do not.
template <class T, int NS, class F>
static void with_tile(const Geo& g, long long copies, F&& f) {
    using Large = GenTile<T, NS, 64, 32, sizeof(T) == 4 ? 8 : 4>;
    using Small = GenTile<T, NS, 32, 16, 4>;
    if (copies * gen_tiles<Large>(g) >= 512)
        f((Large*)nullptr);
    else
        f((Small*)nullptr);
}

hipError_t launch_energy_grad_gen(const Geo& g, const CoefD& kd, bool f64, int batch, const void* m,
                                  const uint8_t* mask, void* grad, void* c, void* F, double* part, int* tiles,
                                  hipStream_t st) {
    if (!kd.gen || kd.gen->ns > GEN_MAX_SHELLS) return hipErrorInvalidValue;
    auto go = [&](auto tc) {
        using T = decltype(tc);
        with_disc<T>(kd, [&](auto& k, auto nsc) {
            constexpr int NS = decltype(nsc)::value;
            using TL = EnergyTile<T, NS>;
            const long long n = gen_tiles<TL>(g), most = LAUNCH_THREADS / TL::NTH;
            *tiles = (int)n;
            for (long long t0 = 0; t0 < batch * n; t0 += most)
                hipLaunchKernelGGL((k_energy_grad_gen<T, NS>), dim3((unsigned)std::min(most, batch * n - t0)),
                                   dim3(TL::NTH), 0, st, g, kd.gen->ns, (int)t0, k, (const T*)m, mask, (T*)grad, (T*)c,
                                   (T*)F, part);
        });
    };
    if (f64)
        go(double(0));
    else
        go(float(0));
    return hipGetLastError();
}

hipError_t launch_tangent_hvp_gen(const Geo& g, const CoefD& kd, bool f64, bool frame, int batch, const void* m,
                                  const void* c, const uint8_t* mask, int nvec, long long vbs, const void* V, void* W,
                                  DoneFlags done, hipStream_t st) {
    if (!kd.gen || kd.gen->ns > GEN_MAX_SHELLS) return hipErrorInvalidValue;
    if (vbs <= 0) vbs = (long long)nvec * (frame ? 2 : 3) * g.N;
    auto go = [&](auto tc, auto fc) {
        using T = decltype(tc);
        constexpr bool FR = decltype(fc)::value;
        with_disc<T>(kd, [&](auto& k, auto nsc) {
            constexpr int NS = decltype(nsc)::value;
            with_tile<T, NS>(g, (long long)batch * nvec, [&](auto tl) {
                using TL = std::remove_pointer_t<decltype(tl)>;
                // vectors a launch
                const long long most = std::max(1LL, LAUNCH_THREADS / (batch * gen_tiles<TL>(g) * TL::NTH));
                for (long long j0 = 0; j0 < nvec; j0 += most) {
                    const int nj = (int)std::min(most, nvec - j0);
                    const size_t o = (size_t)j0 * (FR ? 2 : 3) * g.N;
                    hipLaunchKernelGGL((k_tangent_hvp_gen<T, FR, NS, TL>),
                                       dim3((unsigned)(batch * gen_tiles<TL>(g) * nj)), dim3(TL::NTH), 0, st, g, k,
                                       (const T*)m, (const T*)c, mask, nj, vbs, (const T*)V + o, (T*)W + o, done);
                }
            });
        });
    };
    if (f64) {
        if (frame)
            go(double(0), std::true_type{});
        else
            go(double(0), std::false_type{});
    } else {
        if (frame)
            go(float(0), std::true_type{});
        else
            go(float(0), std::false_type{});
    }
    return hipGetLastError();
}

}  // namespace moto
