// stencil.hip -- lattice kernels: energy/gradient, Euclidean Hessian apply, mixed
// parameter derivatives, topological charge; the entry to the tangent HVP's
// kernels and to those for more than three shells.
//
// Every kernel of the stencil stages a (TX+4) x (TY+4) tile of 3-vectors in LDS
// (periodic wrap at the halo) and evaluates the three-shell sums of the spin
// Hamiltonian (Methods, Eq. param-hamiltonian) at one site per thread.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "kernels.hpp"
#include "tile_ops.hpp"

namespace moto {

// Map a block to (lattice b, tile origin).
struct TileIdx {
    int id, b, tx0, ty0;
};

__device__ __forceinline__ TileIdx tile_of(const Geo& g, int id) {
    TileIdx r;
    r.id = id;
    r.b = id / g.tiles;
    const int t = id - r.b * g.tiles;
    r.tx0 = (t % g.tiles_x) * TX;
    r.ty0 = (t / g.tiles_x) * TY;
    return r;
}

// spins of one tile and its halo (tid: thread among the tile's NT)
template <class T>
__device__ __forceinline__ void stage_spins(TileLDS<T>& t, const Geo& g, const T* __restrict__ mb, int tx0, int ty0,
                                            int tid) {
    const size_t N = g.N;
#pragma unroll
    for (int q = 0; q < (TILE_SITES + NT - 1) / NT; ++q) {
        const int i = tid + q * NT;
        if (i < TILE_SITES) {
            const int ly = i / LXH, lx = i - ly * LXH;
            const int s = wrap1(tx0 + lx - HALO, g.Lx) + g.Lx * wrap1(ty0 + ly - HALO, g.Ly);
            t.u[0][ly][lx] = mb[s];
            t.u[1][ly][lx] = mb[N + s];
            t.u[2][ly][lx] = mb[2 * N + s];
        }
    }
}

// the sums of lattice b in their places: E[b] and
// dtheta[b][.] = (J_0..J_{ns-1}, D_0..D_{ns-1}, K, Bx, By, Bz)
template <int NP>
__device__ __forceinline__ void store_sums(const double (&v)[NP], int b, int ns, double* __restrict__ E,
                                           double* __restrict__ dth) {
    if (E) E[b] = v[0];
    if constexpr (NP == NPART) {
        if (!dth) return;
        double* o = dth + (size_t)b * (2 * ns + 4);
        for (int s = 0; s < ns; ++s) {
            o[s] = v[1 + s];
            o[ns + s] = v[4 + s];
        }
        o[2 * ns] = v[7];
        o[2 * ns + 1] = v[8];
        o[2 * ns + 2] = v[9];
        o[2 * ns + 3] = v[10];
    }
}

// One tile per workgroup; the tile's sums go to part[tile][NP].  Consecutive
// tiles of a lattice run on one XCD, whose L2 then serves the halo rows.
template <class T, int NP>
__global__ __launch_bounds__(NT) void k_energy_grad(Geo g, Coef<T> k, const T* __restrict__ m,
                                                    const uint8_t* __restrict__ mask, T* __restrict__ grad,
                                                    T* __restrict__ cout, T* __restrict__ F,
                                                    double* __restrict__ part) {
    __shared__ TileLDS<T> t;
    __shared__ double red[(NP ? NP : 1) * (NT / 64)];
    const TileIdx ti = tile_of(g, xcd_order(true));
    const size_t off3 = (size_t)ti.b * 3 * g.N, off1 = (size_t)ti.b * g.N;
    stage_spins(t, g, m + off3, ti.tx0, ti.ty0, threadIdx.x);
    __syncthreads();
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    const int x = ti.tx0 + lx, y = ti.ty0 + ly;
    double v[NP ? NP : 1];
#pragma unroll
    for (int q = 0; q < NP; ++q) v[q] = 0.0;
    if (x < g.Lx && y < g.Ly)
        energy_site<T, NP, TX>(t, lx + HALO, ly + HALO, x + g.Lx * y, g, k, mask ? mask + off1 : nullptr,
                           grad ? grad + off3 : nullptr, cout ? cout + off1 : nullptr, F ? F + off3 : nullptr, v);
    if constexpr (NP > 0) {
        block_sum<NP>(v, red);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int q = 0; q < NP; ++q) part[(size_t)ti.id * NP + q] = v[q];
        }
    }
}

// One lattice per workgroup, NT threads for each of its (at most four) tiles:
// the sums stay in the workgroup, so a small lattice is one launch instead of
// two (the second costs the host and the stream about 2 us each).  Three and four
// tiles in large batches take the two launches all the same: with workgroups of
// 768 and 1024 threads few are at hand for a unit that waits, and the LDS of four
// tiles is held by all (us of one launch / two, the energies alone, FP64, 32x32:
// 1024 lattices 15.8 / 14.5, 4096 61 / 46; 512 8.8 / 10.8; one and two tiles gain
// at any batch, 8192 x 64x8 44 / 49).  The results are the same bits.
constexpr int ONE_WG_TILES = 4;
constexpr int ONE_WG_BATCH_TILES = 4096;
template <class T, int NP>
__global__ __launch_bounds__(ONE_WG_TILES * NT) void k_energy_grad_wg(Geo g, Coef<T> k, const T* __restrict__ m,
                                                                      const uint8_t* __restrict__ mask,
                                                                      T* __restrict__ grad, T* __restrict__ cout,
                                                                      T* __restrict__ F, int ns,
                                                                      double* __restrict__ E,
                                                                      double* __restrict__ dth) {
    __shared__ TileLDS<T> t[ONE_WG_TILES];
    constexpr int NV = NP ? NP : 1;
    __shared__ double red[ONE_WG_TILES * NT / 64][NV];
    const int b = blockIdx.x, w = threadIdx.x / NT, tid = threadIdx.x % NT;  // tile w of lattice b
    const int tx0 = (w % g.tiles_x) * TX, ty0 = (w / g.tiles_x) * TY;
    const size_t off3 = (size_t)b * 3 * g.N, off1 = (size_t)b * g.N;
    stage_spins(t[w], g, m + off3, tx0, ty0, tid);
    __syncthreads();
    const int lx = tid % TX, ly = tid / TX;
    const int x = tx0 + lx, y = ty0 + ly;
    double v[NV];
#pragma unroll
    for (int q = 0; q < NP; ++q) v[q] = 0.0;
    if (x < g.Lx && y < g.Ly)
        energy_site<T, NP, TX>(t[w], lx + HALO, ly + HALO, x + g.Lx * y, g, k, mask ? mask + off1 : nullptr,
                           grad ? grad + off3 : nullptr, cout ? cout + off1 : nullptr, F ? F + off3 : nullptr, v);
    if constexpr (NP > 0) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const double s = wave_sum(v[q]);
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = s;
        }
        __syncthreads();
        // added as the two launches do it: a tile's waves one after another, then
        // the butterfly over the tiles
        if (threadIdx.x == 0) {
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                double ts[ONE_WG_TILES];
#pragma unroll
                for (int i = 0; i < ONE_WG_TILES; ++i) {
                    ts[i] = 0.0;
                    if (i < g.tiles)
                        for (int u = 0; u < NT / 64; ++u) ts[i] += red[i * (NT / 64) + u][q];
                }
                v[q] = (ts[0] + ts[2]) + (ts[1] + ts[3]);
            }
            store_sums<NV>(v, b, ns, E, dth);
        }
    }
}

// Mixed derivatives d(g.U)/dtheta as per-block partials in the same slots:
//   [0, -2 U.S_0, -2 U.S_1, -2 U.S_2, 2 U.Q_0, 2 U.Q_1, 2 U.Q_2, -2 U_z m_z, -U_x, -U_y, -U_z]
template <class T>
__global__ __launch_bounds__(NT) void k_param_mixed(Geo g, const T* __restrict__ m, const T* __restrict__ U,
                                                    double* __restrict__ part) {
    __shared__ TileLDS<T> t;
    __shared__ double red[NPART * (NT / 64)];
    const TileIdx ti = tile_of(g, blockIdx.x);
    const size_t off3 = (size_t)ti.b * 3 * g.N;
    const T* mb = m + off3;
    for (int i = threadIdx.x; i < TILE_SITES; i += NT) {
        const int lx = i % LXH, ly = i / LXH;
        const int x = wrapi(ti.tx0 + lx - HALO, g.Lx), y = wrapi(ti.ty0 + ly - HALO, g.Ly);
        const int s = x + g.Lx * y;
        t.u[0][ly][lx] = mb[s];
        t.u[1][ly][lx] = mb[g.N + s];
        t.u[2][ly][lx] = mb[2 * g.N + s];
    }
    __syncthreads();
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    const int x = ti.tx0 + lx, y = ti.ty0 + ly;
    double v[NPART];
#pragma unroll
    for (int q = 0; q < NPART; ++q) v[q] = 0.0;
    if (x < g.Lx && y < g.Ly) {
        const int cx = lx + HALO, cy = ly + HALO;
        const int s = x + g.Lx * y;
        const T* ub = U + off3;
        const T ui[3] = {ub[s], ub[g.N + s], ub[2 * g.N + s]};
        T S[3][3], Q[3][3];
        shell_sums(t, cx, cy, S, Q);
#pragma unroll
        for (int sh = 0; sh < 3; ++sh) {
            v[1 + sh] = -2.0 * ((double)ui[0] * S[sh][0] + (double)ui[1] * S[sh][1] + (double)ui[2] * S[sh][2]);
            v[4 + sh] = 2.0 * ((double)ui[0] * Q[sh][0] + (double)ui[1] * Q[sh][1] + (double)ui[2] * Q[sh][2]);
        }
        v[7] = -2.0 * (double)ui[2] * t.u[2][cy][cx];
        v[8] = -(double)ui[0];
        v[9] = -(double)ui[1];
        v[10] = -(double)ui[2];
    }
    block_sum<NPART>(v, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NPART; ++q) part[(size_t)blockIdx.x * NPART + q] = v[q];
    }
}

// Parameter-weighted gradient sum  out_i = sum_q w_q dg_i/dtheta_q  (the
// adjoint of the parameter partials; g is linear in theta):
//   J_s: -2 S_s,  D_s: 2 Q_s,  K: -2 m_z z,  B_a: -e_a.
// w = [batch][2 ns + 4] (FP64), theta order (J_0.., D_0.., K, Bx, By, Bz).
template <class T>
__global__ __launch_bounds__(NT) void k_param_grad_apply(Geo g, int ns, const T* __restrict__ m,
                                                         const double* __restrict__ w, T* __restrict__ out) {
    __shared__ TileLDS<T> t;
    const TileIdx ti = tile_of(g, blockIdx.x);
    const size_t off3 = (size_t)ti.b * 3 * g.N;
    const T* mb = m + off3;
    for (int i = threadIdx.x; i < TILE_SITES; i += NT) {
        const int lx = i % LXH, ly = i / LXH;
        const int x = wrapi(ti.tx0 + lx - HALO, g.Lx), y = wrapi(ti.ty0 + ly - HALO, g.Ly);
        const int s = x + g.Lx * y;
        t.u[0][ly][lx] = mb[s];
        t.u[1][ly][lx] = mb[g.N + s];
        t.u[2][ly][lx] = mb[2 * g.N + s];
    }
    __syncthreads();
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    const int x = ti.tx0 + lx, y = ti.ty0 + ly;
    if (x >= g.Lx || y >= g.Ly) return;
    const int cx = lx + HALO, cy = ly + HALO;
    const int s = x + g.Lx * y;
    const double* wb = w + (size_t)ti.b * (2 * ns + 4);
    T S[3][3], Q[3][3];
    shell_sums(t, cx, cy, S, Q);
    double o[3];
    for (int c = 0; c < 3; ++c) {
        double v = -wb[2 * ns + 1 + c];
        for (int sh = 0; sh < ns; ++sh) v += -2.0 * wb[sh] * S[sh][c] + 2.0 * wb[ns + sh] * Q[sh][c];
        o[c] = v;
    }
    o[2] += -2.0 * wb[2 * ns] * (double)t.u[2][cy][cx];
    T* ob = out + off3;
    ob[s] = (T)o[0];
    ob[g.N + s] = (T)o[1];
    ob[2 * g.N + s] = (T)o[2];
}

// Fixed-order reduction of the per-tile sums of each lattice.
template <int NP>
__global__ __launch_bounds__(NT) void k_reduce_partials(const double* __restrict__ part, int tiles, int ns,
                                                        double* __restrict__ E, double* __restrict__ dth) {
    __shared__ double red[NP * (NT / 64)];
    const int b = blockIdx.x;
    double v[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) v[q] = 0.0;
    for (int i = threadIdx.x; i < tiles; i += NT) {
        const double* p = part + ((size_t)b * tiles + i) * NP;
#pragma unroll
        for (int q = 0; q < NP; ++q) v[q] += p[q];
    }
    block_sum<NP>(v, red);
    if (threadIdx.x == 0) store_sums<NP>(v, b, ns, E, dth);
}

// Euclidean Hessian apply W_j = A V_j (ambient, unmasked).
template <class T>
__global__ __launch_bounds__(NT) void k_hessian_apply(Geo g, Coef<T> k, int nvec, const T* __restrict__ V,
                                                      T* __restrict__ W) {
    __shared__ TileLDS<T> t;
    const TileIdx ti = tile_of(g, blockIdx.x);
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    const int x = ti.tx0 + lx, y = ti.ty0 + ly;
    const int sc = x + g.Lx * y;
    const size_t vstride = (size_t)3 * g.N;
    for (int j = 0; j < nvec; ++j) {
        const T* vj = V + ((size_t)ti.b * nvec + j) * vstride;
        __syncthreads();
        for (int i = threadIdx.x; i < TILE_SITES; i += NT) {
            const int lx2 = i % LXH, ly2 = i / LXH;
            const int x2 = wrapi(ti.tx0 + lx2 - HALO, g.Lx), y2 = wrapi(ti.ty0 + ly2 - HALO, g.Ly);
            const int s = x2 + g.Lx * y2;
            t.u[0][ly2][lx2] = vj[s];
            t.u[1][ly2][lx2] = vj[g.N + s];
            t.u[2][ly2][lx2] = vj[2 * g.N + s];
        }
        __syncthreads();
        if (x < g.Lx && y < g.Ly) {
            T a[3];
            apply_A_tile(t, lx + HALO, ly + HALO, k, a);
            T* wj = W + ((size_t)ti.b * nvec + j) * vstride;
            wj[sc] = a[0];
            wj[g.N + sc] = a[1];
            wj[2 * g.N + sc] = a[2];
        }
    }
}

// Berg-Luescher charge: per-block partials of -(1/4pi) * sum of the signed
// solid angles of the two triangles (x,y),(x+1,y),(x,y+1) and
// (x+1,y),(x+1,y+1),(x,y+1) of every cell.
__global__ __launch_bounds__(NT) void k_topo_charge(Geo g, const double* __restrict__ m,
                                                    double* __restrict__ part) {
    __shared__ double red[NT / 64];
    const TileIdx ti = tile_of(g, blockIdx.x);
    const double* mb = m + (size_t)ti.b * 3 * g.N;
    const int x = ti.tx0 + threadIdx.x % TX, y = ti.ty0 + threadIdx.x / TX;
    double v[1] = {0.0};
    if (x < g.Lx && y < g.Ly) {
        const int x1 = (x + 1) % g.Lx, y1 = (y + 1) % g.Ly;
        const int s00 = x + g.Lx * y, s10 = x1 + g.Lx * y, s01 = x + g.Lx * y1, s11 = x1 + g.Lx * y1;
        const int tri[2][3] = {{s00, s10, s01}, {s10, s11, s01}};
        double q = 0.0;
        for (int t2 = 0; t2 < 2; ++t2) {
            double a[3], b[3], c[3];
            for (int cc = 0; cc < 3; ++cc) {
                a[cc] = mb[cc * g.N + tri[t2][0]];
                b[cc] = mb[cc * g.N + tri[t2][1]];
                c[cc] = mb[cc * g.N + tri[t2][2]];
            }
            const double bc0 = b[1] * c[2] - b[2] * c[1], bc1 = b[2] * c[0] - b[0] * c[2],
                         bc2 = b[0] * c[1] - b[1] * c[0];
            const double num = a[0] * bc0 + a[1] * bc1 + a[2] * bc2;
            const double den = 1.0 + (a[0] * b[0] + a[1] * b[1] + a[2] * b[2]) +
                               (b[0] * c[0] + b[1] * c[1] + b[2] * c[2]) + (c[0] * a[0] + c[1] * a[1] + c[2] * a[2]);
            q += 2.0 * atan2(num, den);
        }
        v[0] = -q / (4.0 * M_PI);
    }
    block_sum<1>(v, red);
    if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

// --------------------------------------------------------------------------
// Launchers
// --------------------------------------------------------------------------

// sums of every lattice from its per-tile rows of NP
template <int NP>
static void reduce_partials(int tiles, int batch, const double* part, int ns, double* E, double* dth,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_reduce_partials<NP>, dim3(batch), dim3(NT), 0, st, part, tiles, ns, E, dth);
}

template <class T, int NP>
static void go_energy(const Geo& g, const CoefD& kd, int batch, const void* m, const uint8_t* mask, void* grad,
                      void* c, void* F, double* part, int ns, double* E, double* dth, hipStream_t st) {
    const Coef<T> k = coef_cast<T>(kd);
    if (g.tiles <= 2 || (g.tiles <= ONE_WG_TILES && (long long)batch * g.tiles < ONE_WG_BATCH_TILES)) {
        hipLaunchKernelGGL((k_energy_grad_wg<T, NP>), dim3(batch), dim3(NT * g.tiles), 0, st, g, k, (const T*)m, mask,
                           (T*)grad, (T*)c, (T*)F, ns, E, dth);
        return;
    }
    hipLaunchKernelGGL((k_energy_grad<T, NP>), dim3(batch * g.tiles), dim3(NT), 0, st, g, k, (const T*)m, mask,
                       (T*)grad, (T*)c, (T*)F, part);
    if constexpr (NP > 0) reduce_partials<NP>(g.tiles, batch, part, ns, E, dth, st);
}

hipError_t launch_energy_grad(const Geo& g, const CoefD& kd, bool f64, int batch, const void* m,
                              const uint8_t* mask, void* grad, void* c, void* F, double* part, int ns, double* E,
                              double* dth, hipStream_t st) {
    if (kd.gen) {
        if (dth) return hipErrorInvalidValue;
        int tiles = 0;
        const hipError_t e = launch_energy_grad_gen(g, kd, f64, batch, m, mask, grad, c, F, part, &tiles, st);
        if (e != hipSuccess) return e;
        if (E) reduce_partials<1>(tiles, batch, part, ns, E, nullptr, st);
        return hipGetLastError();
    }
    auto go = [&](auto np) {
        constexpr int NP = decltype(np)::value;
        if (f64)
            go_energy<double, NP>(g, kd, batch, m, mask, grad, c, F, part, ns, E, dth, st);
        else
            go_energy<float, NP>(g, kd, batch, m, mask, grad, c, F, part, ns, E, dth, st);
    };
    if (dth)
        go(std::integral_constant<int, NPART>{});
    else if (E)
        go(std::integral_constant<int, 1>{});
    else
        go(std::integral_constant<int, 0>{});
    return hipGetLastError();
}

hipError_t launch_param_mixed(const Geo& g, bool f64, int batch, const void* m, const void* U, double* part, int ns,
                              double* out, hipStream_t st) {
    dim3 grid(batch * g.tiles);
    if (f64)
        hipLaunchKernelGGL(k_param_mixed<double>, grid, dim3(NT), 0, st, g, (const double*)m, (const double*)U,
                           part);
    else
        hipLaunchKernelGGL(k_param_mixed<float>, grid, dim3(NT), 0, st, g, (const float*)m, (const float*)U,
                           part);
    reduce_partials<NPART>(g.tiles, batch, part, ns, nullptr, out, st);
    return hipGetLastError();
}

hipError_t launch_param_grad_apply(const Geo& g, int ns, bool f64, int batch, const void* m, const double* w,
                                  void* out, hipStream_t st) {
    dim3 grid(batch * g.tiles);
    if (f64)
        hipLaunchKernelGGL(k_param_grad_apply<double>, grid, dim3(NT), 0, st, g, ns, (const double*)m, w,
                           (double*)out);
    else
        hipLaunchKernelGGL(k_param_grad_apply<float>, grid, dim3(NT), 0, st, g, ns, (const float*)m, w,
                           (float*)out);
    return hipGetLastError();
}

hipError_t launch_tangent_hvp(const Geo& g, const CoefD& kd, bool f64, bool frame, int batch, const void* m,
                              const void* c, const uint8_t* mask, int nvec, const void* V, void* W,
                              DoneFlags done, hipStream_t st, int variant, long long vbs) {
    if (vbs <= 0) vbs = (long long)nvec * (frame ? 2 : 3) * g.N;
    // lattices a launch: no kernel spends more than four times NT threads on a
    // tile and vector
    const long long most = std::max(1LL, LAUNCH_THREADS / (4LL * NT * g.tiles * nvec));
    const size_t es = f64 ? sizeof(double) : sizeof(float);
    const size_t sm = es * 3 * g.N, sc = es * g.N, sv = es * (size_t)vbs;
    for (long long b0 = 0; b0 < batch; b0 += most) {
        const int nb = (int)std::min(most, batch - b0);
        const void *mb = (const char*)m + sm * b0, *cb = (const char*)c + sc * b0, *Vb = (const char*)V + sv * b0;
        void* Wb = (char*)W + sv * b0;
        const uint8_t* mk = mask ? mask + (size_t)g.N * b0 : nullptr;
        const DoneFlags db(done.p ? done.p + done.stride * b0 : nullptr, done.stride);
        hipError_t e;
        if (kd.gen)
            e = launch_tangent_hvp_gen(g, kd, f64, frame, nb, mb, cb, mk, nvec, vbs, Vb, Wb, db, st);
        else if (frame)
            e = launch_hvp_frame(variant, g, kd, f64, nb, mb, cb, mk, nvec, Vb, Wb, db, st, vbs);
        else
            e = vbs == (long long)nvec * 3 * g.N ? launch_hvp_ambient(g, kd, f64, nb, mb, cb, mk, nvec, Vb, Wb, db, st)
                                                 : hipErrorInvalidValue;
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_hessian_apply(const Geo& g, const CoefD& kd, bool f64, int batch, int nvec, const void* V,
                                void* W, hipStream_t st) {
    dim3 grid(batch * g.tiles);
    if (f64)
        hipLaunchKernelGGL(k_hessian_apply<double>, grid, dim3(NT), 0, st, g, coef_cast<double>(kd), nvec,
                           (const double*)V, (double*)W);
    else
        hipLaunchKernelGGL(k_hessian_apply<float>, grid, dim3(NT), 0, st, g, coef_cast<float>(kd), nvec,
                           (const float*)V, (float*)W);
    return hipGetLastError();
}

hipError_t launch_topo_charge(const Geo& g, int batch, const double* m, double* part, double* Q, hipStream_t st) {
    hipLaunchKernelGGL(k_topo_charge, dim3(batch * g.tiles), dim3(NT), 0, st, g, m, part);
    reduce_partials<1>(g.tiles, batch, part, 0, Q, nullptr, st);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Scratch of the allocation-free energy/gradient entry point: the per-tile
// partial sums live in this file-scope array, one copy per GPU for the life
// of the process.  Host code must not use the array's name as an address (on
// the host it is only a stand-in); energy_scratch() looks up each device's
// copy once, with that device current, and hands out that pointer.
// --------------------------------------------------------------------------
static __device__ __align__(256) double scratch[ENERGY_SCRATCH_BYTES / sizeof(double)];

hipError_t energy_scratch(double** out) {
    constexpr int MAXDEV = 64;
    static std::mutex mu;
    static double* ptr[MAXDEV] = {};
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAXDEV) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr[dev] = (double*)p;
    }
    *out = ptr[dev];
    return hipSuccess;
}

}  // namespace moto
