// step.hip -- device kernels of the outer layer: reflected force and one
// L-BFGS / fixed / nonlinear-CG rotation step of every spin (Results,
// "Bilayer MMF": L-BFGS and CG are the paper's two outer optimisers;
// Supplementary Note 1, Algorithm 1, bilayer loop).
//
// The L-BFGS two-loop recursion is run in coefficient space: every vector it
// touches is a combination of the stored pairs S_j, Y_j and the current G, so
// one fused pass computes the Gram matrix of {S_0.., Y_0.., G} (after the
// projection transport of the stored pairs), one workgroup sums its
// partials and runs the recursion on that small matrix, and one pass forms the direction.
#include "dense_wg.hpp"
#include "kernels.hpp"

namespace moto {

constexpr int SMEM = 16;                  // max L-BFGS memory
constexpr int SNV = 2 * SMEM + 1;         // max Gram basis size
constexpr int SNE = SNV * (SNV + 1) / 2;  // Gram entries (upper triangle)
constexpr int SPART = SNE + 1;            // + ||F_mmf||^2
constexpr int SCH = 64;                   // sites per staged chunk
constexpr int MAXR = 4;                   // max reflected modes

struct StepHdr {
    int count, head, have_prev, stopped;
    int iters;
    int cu;  // number of pairs the coefficients below refer to (G is coef[2*cu])
    int pad1, pad2;
    double fnorm;
    double cg_c;  // CG: the step taken last time = cg_c x its direction
    double coef[SNV];
};

constexpr int CG_RESTART = 50;  // CG restart period (steps)

struct StepPtrs {
    StepHdr* hdr;
    double *S, *Y, *G, *Gp, *dp, *d, *pgram, *pdot, *pmax;
    size_t vstride;  // doubles between stored vectors
    int nblk;
};

static size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

static int step_blocks(int N) {
    int nb = (N + SCH - 1) / SCH;
    return nb < 256 ? nb : 256;
}

static StepPtrs step_ptrs(void* state, int N, int mem, size_t* total) {
    StepPtrs P;
    char* base = (char*)state;
    const int nblk = step_blocks(N);
    const size_t v = al(sizeof(double) * 3 * (size_t)N);
    size_t o = 0;
    P.hdr = (StepHdr*)(base + o);
    o += al(sizeof(StepHdr));
    P.S = (double*)(base + o);
    o += v * mem;
    P.Y = (double*)(base + o);
    o += v * mem;
    P.G = (double*)(base + o);
    o += v;
    P.Gp = (double*)(base + o);
    o += v;
    P.dp = (double*)(base + o);
    o += v;
    P.d = (double*)(base + o);
    o += v;
    P.pgram = (double*)(base + o);
    o += al(sizeof(double) * SPART * nblk);
    P.pdot = (double*)(base + o);
    o += al(sizeof(double) * MAXR * nblk);
    P.pmax = (double*)(base + o);
    o += al(sizeof(double) * nblk);
    P.vstride = v / sizeof(double);
    P.nblk = nblk;
    if (total) *total = o;
    return P;
}

size_t step_state_bytes(int N, int mem) {
    size_t t = 0;
    step_ptrs(nullptr, N, mem, &t);
    return t;
}

// Ring bookkeeping shared by the Gram and control kernels: the pair formed
// at this step goes to `slot`; logical pair j (oldest first) lives in
// physical slot (h_new + j) % mem.
struct Ring {
    int c_new, h_new, slot;
};

// slot of logical pair j < mem (a division would cost 40 instructions)
__device__ __forceinline__ int ring_slot(int head, int j, int mem) {
    const int q = head + j;
    return q >= mem ? q - mem : q;
}

__device__ __forceinline__ Ring ring_next(const StepHdr* h, int mem, int rule) {
    Ring r;
    r.slot = -1;
    r.c_new = h->count;
    r.h_new = h->head;
    if (h->have_prev && (rule == 0 || rule == 2)) {
        if (h->count < mem) {
            r.slot = ring_slot(h->head, h->count, mem);
            r.c_new = h->count + 1;
        } else {
            r.slot = h->head;
            r.h_new = ring_slot(h->head, 1, mem);
        }
    }
    return r;
}

// Members of a population stepped by one launch: member y = blockIdx.y owns
// the step state at + y sb bytes, spins and forces at + y m3 doubles and its
// modes at + y v3 doubles (all zero for a single search).
struct StepBatch {
    long long sb = 0, m3 = 0, v3 = 0;
};

__device__ __forceinline__ StepPtrs member_ptrs(StepPtrs P, const StepBatch& B) {
    const long long off = (long long)blockIdx.y * B.sb;
    auto sh = [&](auto* q) { return reinterpret_cast<decltype(q)>(reinterpret_cast<char*>(q) + off); };
    P.hdr = sh(P.hdr);
    P.S = sh(P.S);
    P.Y = sh(P.Y);
    P.G = sh(P.G);
    P.Gp = sh(P.Gp);
    P.dp = sh(P.dp);
    P.d = sh(P.d);
    P.pgram = sh(P.pgram);
    P.pdot = sh(P.pdot);
    P.pmax = sh(P.pmax);
    return P;
}

// (1) per-block partial dots F . v_r
__global__ __launch_bounds__(NT) void k_step_dots(StepArgs a, const double* __restrict__ F,
                                                  const double* __restrict__ V, StepPtrs P, StepBatch B) {
    P = member_ptrs(P, B);
    F += blockIdx.y * B.m3;
    V += blockIdx.y * B.v3;
    if (P.hdr->stopped) return;
    __shared__ double red[MAXR * (NT / 64)];
    double v[MAXR] = {0, 0, 0, 0};
    const size_t n3 = 3 * (size_t)a.N;
    const int per = (a.N + gridDim.x - 1) / gridDim.x;
    const int s0 = blockIdx.x * per, s1 = min(a.N, s0 + per);
    for (int s = s0 + threadIdx.x; s < s1; s += NT)
        for (int r = 0; r < a.k_reflect; ++r)
            for (int c = 0; c < 3; ++c) v[r] += F[c * a.N + s] * V[r * n3 + c * a.N + s];
    block_sum<MAXR>(v, red);
    if (threadIdx.x == 0)
        for (int r = 0; r < MAXR; ++r) P.pdot[(size_t)blockIdx.x * MAXR + r] = v[r];
}

// (2) G = -(F - 2 sum_r (F.v_r) v_r); projection transport of the stored
// pairs onto the tangent spaces at m; new pair s = P d_prev, y = G - P G_prev;
// Gram partials of {S_0..S_{c-1}, Y_0..Y_{c-1}, G} and ||F_mmf||^2.
//
// At 128x128 a workgroup has one chunk of sites, and the kernel is a chain of
// latencies: header, partial dots, site loads, transport, Gram.  Every wave takes
// one stored pair (of up to eight), all its loads are issued before the dots are
// summed (those of the next chunk before the Gram of this one), and eight lanes
// share a 2 x 2 tile of Gram entries, each over an eighth of the sites, so that
// four reads from LDS serve four products.  128x128, mean of sixteen steps from
// an empty history: 9.4 -> 8.7 us (12.5 -> 11.9 with 8 pairs).
constexpr int GNT = 512;              // threads
constexpr int GW = GNT / SCH;         // waves
constexpr int GJ = SMEM / GW;         // stored pairs of a wave
constexpr int GH = (SNV + 1) / 2;     // tile rows of the Gram
constexpr int GRG = 8;                // lanes (groups of sites) to a tile
constexpr int GQ = (GH * (GH + 1) / 2 * GRG + GNT - 1) / GNT;  // tiles of a lane
__global__ __launch_bounds__(GNT) void k_step_gram(StepArgs a, const double* __restrict__ m,
                                                   const double* __restrict__ F, const double* __restrict__ V,
                                                   StepPtrs P, StepBatch B) {
    P = member_ptrs(P, B);
    m += blockIdx.y * B.m3;
    F += blockIdx.y * B.m3;
    V += blockIdx.y * B.v3;
    const StepHdr* h = P.hdr;
    if (h->stopped) return;
    __shared__ double fr[MAXR];
    // rows padded by two doubles (16-byte aligned): the lanes of a wave read
    // different vectors at the same site, all on one LDS bank otherwise
    constexpr int SCHP = SCH + 2;
    __shared__ double stage[2 * GH][3][SCHP];
    const Ring rg = ring_next(h, a.mem, a.rule);
    const int c = rg.c_new;
    const int nv = 2 * c + 1;
    const size_t N = a.N, n3 = 3 * N;
    const int nchunks = (a.N + SCH - 1) / SCH;
    // the waves stage the same SCH sites: each forms the site's reflected force,
    // gradient and new pair and transports every GW-th stored pair (wave 0 also
    // writes G, the gradient column and |F|^2)
    static_assert(SCH == WL && SMEM % GW == 0, "one site per lane, whole waves");
    const int t = threadIdx.x % SCH, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / SCH);
    double mi[3], f[3], vr[MAXR][3], dpv[3], gpv[3], sv[GJ][3], yv[GJ][3];
    auto load = [&](int ch) {
        const size_t s = (size_t)ch * SCH + t;
        const bool on = s < N;
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            const size_t o = cc * N + s;
            mi[cc] = on ? m[o] : 0.0;
            f[cc] = on ? F[o] : 0.0;
            dpv[cc] = on && rg.slot >= 0 ? P.dp[o] : 0.0;
            gpv[cc] = on && rg.slot >= 0 ? P.Gp[o] : 0.0;
#pragma unroll
            for (int r = 0; r < MAXR; ++r) vr[r][cc] = on && r < a.k_reflect ? V[r * n3 + o] : 0.0;
#pragma unroll
            for (int q = 0; q < GJ; ++q) {
                const int j = wv + GW * q, ph = ring_slot(rg.h_new, j, a.mem);
                const bool st = on && j < c && ph != rg.slot;
                sv[q][cc] = st ? P.S[ph * P.vstride + o] : 0.0;
                yv[q][cc] = st ? P.Y[ph * P.vstride + o] : 0.0;
            }
        }
    };
    if ((int)blockIdx.x < nchunks) load(blockIdx.x);
    // fr[r] = sum over the blocks' partials: wave r, lanes over the blocks
    static_assert(MAXR <= GW, "a wave per reflected mode");
    if (wv < MAXR) {
        double s = 0.0;
        if (wv < a.k_reflect)
            for (int b = t; b < P.nblk; b += WL) s += P.pdot[(size_t)b * MAXR + wv];
        s = wave_sum(s);
        if (t == 0) fr[wv] = s;
    }
    // tiles of this lane (upper triangle) and its group of sites
    const int hn = c + 1, g = threadIdx.x % GRG;
    int ti[GQ], tj[GQ];
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
        int p = (int)threadIdx.x / GRG + q * (GNT / GRG), i = 0;
        if (p < hn * (hn + 1) / 2) {
            while (p >= hn - i) {
                p -= hn - i;
                ++i;
            }
            ti[q] = i;
            tj[q] = i + p;
        } else {
            ti[q] = -1;
            tj[q] = 0;
        }
    }
    double acc[GQ][2][2], fn2 = 0.0;
#pragma unroll
    for (int q = 0; q < GQ; ++q) acc[q][0][0] = acc[q][0][1] = acc[q][1][0] = acc[q][1][1] = 0.0;
    for (int ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        __syncthreads();
        {
            const size_t s = (size_t)ch * SCH + t;
            const bool on = s < N;
            double gr[3];
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                double v = f[cc];
#pragma unroll
                for (int r = 0; r < MAXR; ++r)
                    if (r < a.k_reflect) v -= 2.0 * fr[r] * vr[r][cc];
                if (wv == 0) {
                    fn2 += v * v;
                    if (on) P.G[cc * N + s] = -v;
                    stage[2 * c][cc][t] = -v;
                }
                gr[cc] = -v;
            }
            auto project = [&](double (&x)[3]) {  // onto the tangent space at m
                const double d = mi[0] * x[0] + mi[1] * x[1] + mi[2] * x[2];
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) x[cc] -= d * mi[cc];
            };
#pragma unroll
            for (int q = 0; q < GJ; ++q) {
                const int j = wv + GW * q;
                if (j >= c) break;
                const int ph = ring_slot(rg.h_new, j, a.mem);
                const bool fresh = ph == rg.slot;
                if (fresh) {
#pragma unroll
                    for (int cc = 0; cc < 3; ++cc) {
                        sv[q][cc] = dpv[cc];
                        yv[q][cc] = gpv[cc];
                    }
                }
                project(sv[q]);
                project(yv[q]);
                double* Sj = P.S + ph * P.vstride;
                double* Yj = P.Y + ph * P.vstride;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    if (fresh) yv[q][cc] = gr[cc] - yv[q][cc];
                    if (on) {
                        Sj[cc * N + s] = sv[q][cc];
                        Yj[cc * N + s] = yv[q][cc];
                    }
                    stage[j][cc][t] = sv[q][cc];
                    stage[c + j][cc][t] = yv[q][cc];
                }
            }
        }
        if (ch + (int)gridDim.x < nchunks) load(ch + gridDim.x);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
            if (ti[q] < 0) continue;
            const double* x = &stage[2 * ti[q]][0][g];
            const double* y = &stage[2 * tj[q]][0][g];
#pragma unroll 2  // all eight steps at once spill
            for (int tt = 0; tt < SCH; tt += GRG)
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    const int o = cc * SCHP + tt;
                    const double x0 = x[o], x1 = x[3 * SCHP + o], y0 = y[o], y1 = y[3 * SCHP + o];
                    acc[q][0][0] += x0 * y0;
                    acc[q][0][1] += x0 * y1;
                    acc[q][1][0] += x1 * y0;
                    acc[q][1][1] += x1 * y1;
                }
        }
    }
    double* pg = P.pgram + (size_t)blockIdx.x * SPART;
    // the tile's lanes are added up; lane g < 4 stores entry (g / 2, g % 2)
#pragma unroll
    for (int q = 0; q < GQ; ++q) {
        double e[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                double v = acc[q][u][z];
                v += dpp_f64<0xB1>(v);
                v += dpp_f64<0x4E>(v);
                v += dpp_f64<0x141>(v);
                e[u][z] = v;
            }
        const int i = 2 * ti[q] + (g >> 1), j = 2 * tj[q] + (g & 1);
        const double v = g == 0 ? e[0][0] : g == 1 ? e[0][1] : g == 2 ? e[1][0] : e[1][1];
        if (ti[q] >= 0 && g < 4 && i <= j && j < nv) pg[i * nv - i * (i - 1) / 2 + (j - i)] = v;
    }
    if (wv == 0) {
        fn2 = wave_sum(fn2);
        if (t == 0) pg[nv * (nv + 1) / 2] = fn2;
    }
}

// (3) Gram of the step basis summed over the blocks, then on one wavefront:
// stop test, two-loop recursion in coefficient space, reset test; writes the
// direction coefficients and the step's outcome.
//
// Both halves are latency: one workgroup reads the blocks' partial rows
// (256 x 154 doubles at 128x128 with 8 pairs), and the recursion is serial in
// the pairs.  A lane takes two neighbouring entries and walks the rows
// (coalesced, sixteen loads in flight, the rows split over the waves that the
// entries leave free).  In the recursion lane j holds S_j . q and Y_j . r, which
// change with each pair by one Gram column, so that a pair costs a lane read and
// two multiply-adds instead of a dot product over the basis.  128x128, mean of
// sixteen steps from an empty history: 45 us with a wave per entry and the
// recursion on one thread, 9.0 with an entry a lane and the dot products, now 7.8
// (10.6 with 8 pairs).
constexpr int CTN = 1024;  // threads
// two entries of a row; the caller's state may be aligned to doubles only
typedef double pair8 __attribute__((ext_vector_type(2), aligned(8)));
__global__ __launch_bounds__(CTN) void k_step_ctrl(StepArgs a, StepPtrs P, double* __restrict__ out, StepBatch B) {
    P = member_ptrs(P, B);
    out += 2 * blockIdx.y;
    StepHdr* h = P.hdr;
    if (h->stopped) {
        if (threadIdx.x == 0) {
            out[0] = h->fnorm;
            out[1] = 1.0;
        }
        return;
    }
    constexpr int WE = 2 * WL;  // entries of a wave
    __shared__ double2 ps[CTN];
    __shared__ double Gm[SNV][SNV];
    __shared__ double fn2;
    const Ring rg = ring_next(h, a.mem, a.rule);
    const int c = rg.c_new;
    const int nv = 2 * c + 1;
    const int ne = nv * (nv + 1) / 2;  // and one more: |F_mmf|^2
    const int lane = wlane(), wv = threadIdx.x / WL;
    static_assert((SPART + WE - 1) / WE <= CTN / WL && SPART <= CTN, "waves for all entries, a thread for each");
    const int chunks = (ne + WE) / WE, parts = (CTN / WL) / chunks;
    const int chunk = wv % chunks, part = wv / chunks;
    {
        const int e = chunk * WE + 2 * lane;
        double2 s = {0.0, 0.0};
        if (part < parts && e <= ne) {
            const double* pg = P.pgram + e;
            constexpr int U = 16;  // rows in flight
            for (int b0 = part; b0 < P.nblk; b0 += U * parts) {
                pair8 x[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    x[u] = *(const pair8*)(pg + (size_t)min(b0 + u * parts, P.nblk - 1) * SPART);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool in = b0 + u * parts < P.nblk;
                    s.x += in ? x[u].x : 0.0;
                    s.y += in ? x[u].y : 0.0;
                }
            }
        }
        ps[threadIdx.x] = s;  // wave wv = part * chunks + chunk
    }
    int gi = 0, gj = threadIdx.x;  // the entry's row and column
    while (gi < nv && gj >= nv - gi) {
        gj -= nv - gi;
        ++gi;
    }
    gj += gi;
    __syncthreads();
    if ((int)threadIdx.x <= ne) {
        const double* pe = (const double*)ps + threadIdx.x;
        double s = 0.0;
        for (int q = 0; q < parts; ++q) s += pe[q * chunks * WE];
        if ((int)threadIdx.x == ne) {
            fn2 = s;
        } else {
            Gm[gi][gj] = s;
            Gm[gj][gi] = s;
        }
    }
    __syncthreads();
    if (threadIdx.x >= WL) return;
    const double fn = sqrt(fn2);
    const bool move = fn > a.tau_F;  // else converged (or NaN)
    if (lane == 0) {
        h->fnorm = fn;
        h->count = c;
        h->head = rg.h_new;
        out[0] = fn;
        out[1] = move ? 0.0 : 1.0;
        if (!move) h->stopped = 1;
    }
    if (!move) return;
    const int iG = 2 * c;
    const bool in = lane < nv;
    // lane i: coefficient of vector i
    double coef = 0.0;
    bool reset = (a.rule == 1);
    if (a.rule == 2) {
        // nonlinear CG (Fletcher-Reeves) on G with one stored pair: S_0 is
        // the transported last step = cg_c x the transported last direction,
        // Y_0 = G - P G_prev, so |P G_prev|^2 = G.G - 2 G.Y_0 + Y_0.Y_0
        if (lane == iG) coef = -a.alpha0;
        if (c >= 1 && h->iters % CG_RESTART != 0) {
            const double GG = Gm[iG][iG], Gy = Gm[c][iG], yy = Gm[c][c];
            const double gpgp = GG - 2.0 * Gy + yy;
            const double beta = gpgp > 0.0 ? GG / gpgp : 0.0;
            const double bs = beta / h->cg_c;
            if (-GG + bs * Gm[0][iG] < 0.0 && lane == 0) coef = a.alpha0 * bs;
        }
    } else if (a.rule == 0) {
        // q = G - sum_i alpha_i Y_i (newest pair first), r = gamma q + sum_i
        // (alpha_i - beta_i) S_i (oldest first); lane j: pair j
        const int j = lane < c ? lane : 0;
        double sy[SMEM], yy[SMEM], ys[SMEM];  // S_j . Y_i, Y_j . Y_i, Y_j . S_i
#pragma unroll
        for (int i = 0; i < SMEM; ++i) {
            sy[i] = i < c ? Gm[j][c + i] : 0.0;
            yy[i] = i < c ? Gm[c + j][c + i] : 0.0;
            ys[i] = i < c ? Gm[c + j][i] : 0.0;
        }
        const double syj = lane < c ? Gm[j][c + j] : 0.0;
        const bool valid = lane < c && syj > a.sy_min;
        const double rho = valid ? 1.0 / syj : 0.0;
        const unsigned long long vm = __ballot(valid);
        double tq = Gm[j][iG], u = Gm[c + j][iG], alph = 0.0, del = 0.0;
#pragma unroll
        for (int i = SMEM - 1; i >= 0; --i) {
            if (!((vm >> i) & 1ull)) continue;
            const double al = rdlane(rho * tq, i);
            if (lane == i) alph = al;
            tq -= al * sy[i];
            u -= al * yy[i];
        }
        const int newest = vm ? 63 - __clzll((long long)vm) : -1;
        const double gamma = newest >= 0 ? Gm[newest][c + newest] / Gm[c + newest][c + newest] : a.alpha0;
        u *= gamma;
#pragma unroll
        for (int i = 0; i < SMEM; ++i) {
            if (!((vm >> i) & 1ull)) continue;
            const double de = rdlane(alph - rho * u, i);
            if (lane == i) del = de;
            u += de * ys[i];
        }
        // coefficients: -del of S_j, gamma alpha of Y_j, -gamma of G
        const double ay = __shfl(alph, lane >= c && lane < iG ? lane - c : 0, WL);
        coef = lane < c ? -del : lane < iG ? gamma * ay : lane == iG ? -gamma : 0.0;
        const double dG = wsum_dpp(in ? coef * Gm[lane][iG] : 0.0);
        if (!(dG < 0.0)) reset = true;
    }
    if (reset) coef = lane == iG ? -a.alpha0 : 0.0;
    if (lane < SNV) h->coef[lane] = coef;
    if (lane == 0) {
        if (reset && a.rule == 0) h->count = 0;
        h->cu = c;
        h->have_prev = 1;
        h->iters += 1;
    }
}

// Threads of the site kernels below: a wave to a workgroup while the blocks
// then cover the lattice (each of the 256 compute units gets its share of the
// latency), whole workgroups beyond.
static int site_threads(int N, int nblk) { return N <= WL * nblk ? WL : NT; }

__device__ __forceinline__ double block_max(double v, double* red /* [NT/64] */) {
    v = wave_max(v);
    if (blockDim.x == WL) return v;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// (4) direction d = P(sum coef . vectors) and per-block max |d_i|.  The pairs
// are read four at a time, all loads in flight (one pair after another: 5.7
// us a call at 128x128 with 8 pairs).
__global__ __launch_bounds__(NT) void k_step_dir(StepArgs a, const double* __restrict__ m, StepPtrs P,
                                                 StepBatch B) {
    P = member_ptrs(P, B);
    m += blockIdx.y * B.m3;
    const StepHdr* h = P.hdr;
    if (h->stopped) return;
    __shared__ double red[NT / 64];
    const int cu = h->cu, head = h->head;
    const size_t N = a.N;
    double mx = 0.0;
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < a.N; s += gridDim.x * blockDim.x) {
        double d[3] = {0.0, 0.0, 0.0};
        constexpr int JU = 4;
        for (int j0 = 0; j0 < cu; j0 += JU) {
            double sv[JU][3], yv[JU][3];
#pragma unroll
            for (int q = 0; q < JU; ++q) {
                const int j = min(j0 + q, cu - 1);
                const size_t o = ring_slot(head, j, a.mem) * P.vstride + s;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    sv[q][cc] = P.S[o + cc * N];
                    yv[q][cc] = P.Y[o + cc * N];
                }
            }
#pragma unroll
            for (int q = 0; q < JU; ++q) {
                if (j0 + q >= cu) break;
                const double cs = h->coef[j0 + q], cy = h->coef[cu + j0 + q];
                if (cs == 0.0 && cy == 0.0) continue;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) d[cc] += cs * sv[q][cc] + cy * yv[q][cc];
            }
        }
        const double cg = h->coef[2 * cu];
        for (int cc = 0; cc < 3; ++cc) d[cc] += cg * P.G[cc * N + s];
        const double mi[3] = {m[s], m[N + s], m[2 * N + s]};
        const double md = mi[0] * d[0] + mi[1] * d[1] + mi[2] * d[2];
        double n2 = 0.0;
        for (int cc = 0; cc < 3; ++cc) {
            d[cc] -= md * mi[cc];
            P.d[cc * N + s] = d[cc];
            n2 += d[cc] * d[cc];
        }
        mx = fmax(mx, sqrt(n2));
    }
    mx = block_max(mx, red);
    if (threadIdx.x == 0) P.pmax[blockIdx.x] = mx;
}

// (5) rotation cap and exponential-map rotation of every spin; d -> d_prev,
// G -> G_prev.  The first site's loads are in flight under the reduction of the
// blocks' largest angles (128x128: 5.2 -> 4.3 us).
__global__ __launch_bounds__(NT) void k_step_rot(StepArgs a, double* __restrict__ m, StepPtrs P, int nblk_dir,
                                                 StepBatch B) {
    P = member_ptrs(P, B);
    m += blockIdx.y * B.m3;
    const StepHdr* h = P.hdr;
    if (h->stopped) return;
    __shared__ double scale_s;
    const int step = gridDim.x * blockDim.x;
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    double d[3], mi[3], g[3];
    auto load = [&]() {  // the first site's before the reduction below
        if (s >= a.N) return;
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            d[cc] = P.d[cc * (size_t)a.N + s];
            mi[cc] = m[cc * (size_t)a.N + s];
            g[cc] = P.G[cc * (size_t)a.N + s];
        }
    };
    load();
    if (threadIdx.x < 64) {  // largest per-site angle over the blocks' partials (wave 0)
        double mx = 0.0;
        for (int b = threadIdx.x; b < nblk_dir; b += 64) mx = fmax(mx, P.pmax[b]);
        mx = wave_max(mx);
        if (threadIdx.x == 0) scale_s = mx > a.theta_max ? a.theta_max / mx : 1.0;
    }
    __syncthreads();
    const double sc = scale_s;
    if (a.rule == 2 && blockIdx.x == 0 && threadIdx.x == 0) P.hdr->cg_c = a.alpha0 * sc;
    while (s < a.N) {
        double n2 = 0.0;
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            d[cc] *= sc;
            n2 += d[cc] * d[cc];
            P.dp[cc * (size_t)a.N + s] = d[cc];
            P.Gp[cc * (size_t)a.N + s] = g[cc];
        }
        const double th = sqrt(n2);
        if (th > 0.0) {
            double ct, st;
            sincos(th, &st, &ct);
            st /= th;
            double o[3], on = 0.0;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                o[cc] = ct * mi[cc] + st * d[cc];
                on += o[cc] * o[cc];
            }
            const double inv = 1.0 / sqrt(on);
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) m[cc * (size_t)a.N + s] = o[cc] * inv;
        }
        s += step;
        load();
    }
}

static hipError_t launch_step_members(const StepArgs& a, double* m, const double* F, const double* V, void* state,
                                      double* out, int members, const StepBatch& B, hipStream_t st) {
    StepPtrs P = step_ptrs(state, a.N, a.mem, nullptr);
    const int nb = P.nblk;
    if (a.k_reflect > 0) hipLaunchKernelGGL(k_step_dots, dim3(nb, members), dim3(NT), 0, st, a, F, V, P, B);
    hipLaunchKernelGGL(k_step_gram, dim3(nb, members), dim3(GNT), 0, st, a, m, F, V, P, B);
    hipLaunchKernelGGL(k_step_ctrl, dim3(1, members), dim3(CTN), 0, st, a, P, out, B);
    const int nt = site_threads(a.N, nb);
    hipLaunchKernelGGL(k_step_dir, dim3(nb, members), dim3(nt), 0, st, a, m, P, B);
    hipLaunchKernelGGL(k_step_rot, dim3(nb, members), dim3(nt), 0, st, a, m, P, nb, B);
    return hipGetLastError();
}

hipError_t launch_step(const StepArgs& a, double* m, const double* F, const double* V, void* state, double* out,
                       hipStream_t st) {
    return launch_step_members(a, m, F, V, state, out, 1, StepBatch{}, st);
}

// One step of P members in one set of launches (member y: spins and forces at
// + y 3N, modes at + y k 3N, step state at + y state_bytes, output at + 2y);
// members whose state says stopped are left alone.
hipError_t launch_step_population(const StepArgs& a, int P, int k, double* m, const double* F, const double* V,
                                  void* state, size_t state_bytes, double* out, hipStream_t st) {
    StepBatch B;
    B.sb = (long long)state_bytes;
    B.m3 = 3LL * a.N;
    B.v3 = (long long)k * 3LL * a.N;
    return launch_step_members(a, m, F, V, state, out, P, B, st);
}

__global__ void k_step_stop(StepHdr* h) {
    if (threadIdx.x == 0) h->stopped = 1;
}

// Marks member y's step state stopped (a member whose eigen-solve failed).
hipError_t launch_step_stop(void* state, int N, int mem, size_t state_bytes, int y, hipStream_t st) {
    StepPtrs P = step_ptrs((char*)state + state_bytes * (size_t)y, N, mem, nullptr);
    hipLaunchKernelGGL(k_step_stop, dim3(1), dim3(64), 0, st, P.hdr);
    return hipGetLastError();
}

// ---- descent seed: m <- R(m, scale * v1 / max_i |v1_i|) ----
__global__ __launch_bounds__(NT) void k_maxnorm(int N, const double* __restrict__ v, double* __restrict__ part) {
    __shared__ double red[NT / 64];
    double mx = 0.0;
    for (int s = blockIdx.x * NT + threadIdx.x; s < N; s += gridDim.x * NT)
        mx = fmax(mx, sqrt(v[s] * v[s] + v[N + s] * v[N + s] + v[2 * N + s] * v[2 * N + s]));
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

__global__ __launch_bounds__(NT) void k_seed_rot(int N, double* __restrict__ m, const double* __restrict__ v,
                                                 double sse, const double* __restrict__ part, int nblk) {
    __shared__ double sc;
    if (threadIdx.x < 64) {  // largest partial (wave 0)
        double mx = 0.0;
        for (int b = threadIdx.x; b < nblk; b += 64) mx = fmax(mx, part[b]);
        mx = wave_max(mx);
        if (threadIdx.x == 0) sc = mx > 0.0 ? sse / mx : 0.0;
    }
    __syncthreads();
    for (int s = blockIdx.x * NT + threadIdx.x; s < N; s += gridDim.x * NT) {
        double d[3], mi[3], n2 = 0.0;
        for (int cc = 0; cc < 3; ++cc) {
            d[cc] = sc * v[cc * N + s];
            mi[cc] = m[cc * N + s];
            n2 += d[cc] * d[cc];
        }
        const double th = sqrt(n2);
        if (th > 0.0) {
            const double ct = cos(th), st = sin(th) / th;
            double o[3], on = 0.0;
            for (int cc = 0; cc < 3; ++cc) {
                o[cc] = ct * mi[cc] + st * d[cc];
                on += o[cc] * o[cc];
            }
            const double inv = 1.0 / sqrt(on);
            for (int cc = 0; cc < 3; ++cc) m[cc * N + s] = o[cc] * inv;
        }
    }
}

hipError_t launch_seed_rotate(int N, double* m, const double* v1, double scale_sign_eta, double* part,
                              hipStream_t st) {
    int nb = (N + NT - 1) / NT;
    nb = nb < 256 ? nb : 256;
    hipLaunchKernelGGL(k_maxnorm, dim3(nb), dim3(NT), 0, st, N, v1, part);
    hipLaunchKernelGGL(k_seed_rot, dim3(nb), dim3(NT), 0, st, N, m, v1, scale_sign_eta, part, nb);
    return hipGetLastError();
}

__global__ void k_f64_to_f32(const double* __restrict__ s, float* __restrict__ d, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) d[i] = (float)s[i];
}

hipError_t launch_f64_to_f32(const double* src, float* dst, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_f64_to_f32, dim3((unsigned)((n + NT - 1) / NT)), dim3(NT), 0, st, src, dst, n);
    return hipGetLastError();
}

__global__ void k_mask_zero(double* __restrict__ v, const uint8_t* __restrict__ mask, int N, int ncomp) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= N || mask[s]) return;
    for (int c = 0; c < ncomp; ++c) v[(size_t)c * N + s] = 0.0;
}

// zero fill of a byte range in 16-byte words (buffers are 256-byte aligned);
// a kernel rather than a memset so that the drivers stay graph-capturable
__global__ __launch_bounds__(NT) void k_zero(uint4* __restrict__ p, size_t n16) {
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n16; i += (size_t)gridDim.x * NT) p[i] = z;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st) {
    if (bytes % 16 != 0 || ((uintptr_t)p & 15) != 0) return hipErrorInvalidValue;
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const size_t nb = (n16 + NT - 1) / NT;
    hipLaunchKernelGGL(k_zero, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(NT), 0, st, (uint4*)p, n16);
    return hipGetLastError();
}

// The descent's outcome assembled on the device (MOTO_ASYNC): stop flag and
// ||F|| from the step output, steps taken from the step state, energy and
// lambda_1 (Eo[0], Eo[1]) and the charge Q.
__global__ void k_descend_result(StepPtrs P, const double* __restrict__ out, const double* __restrict__ Eo,
                                 const double* __restrict__ Q, moto_descend_result* __restrict__ res) {
    if (threadIdx.x != 0) return;
    moto_descend_result r;
    r.converged = out[1] != 0.0 ? 1 : 0;
    r.iters = P.hdr->iters;
    r.E = Eo[0];
    r.Q = Q[0];
    r.fnorm = out[0];
    r.lambda1 = Eo[1];
    *res = r;
}

hipError_t launch_descend_result(void* state, int N, int mem, const double* out, const double* Eo, const double* Q,
                                 moto_descend_result* res, hipStream_t st) {
    StepPtrs P = step_ptrs(state, N, mem, nullptr);
    hipLaunchKernelGGL(k_descend_result, dim3(1), dim3(64), 0, st, P, out, Eo, Q, res);
    return hipGetLastError();
}

hipError_t launch_mask_zero(double* v, const uint8_t* mask, int N, int ncomp, hipStream_t st) {
    hipLaunchKernelGGL(k_mask_zero, dim3((N + NT - 1) / NT), dim3(NT), 0, st, v, mask, N, ncomp);
    return hipGetLastError();
}

}  // namespace moto
