// sip.hip -- the strongly implicit procedure for K phi = rho (the preconditioner option
// CPS_PRECOND_SIP).
//
// The paper solves its preconditioned system K phi = rho (Sec. 3.3) with the modified strongly
// implicit procedure of its ref. 24, whose recurrences it does not give.  This is the strongly
// implicit procedure in its original form: Stone's partial-cancellation incomplete
// factorisation M = L U of the 7-point K, extended to three dimensions.  Unknowns are ordered
// lexicographically (x fastest).  L has b, c, d at the -z, -y, -x neighbours (B, S, W) and e
// on the diagonal; U has a unit diagonal and f, g, h at the +x, +y, +z neighbours (E, N, T).
// The six positions where L U fills in beyond K's stencil hold X1 = b f_B, X2 = b g_B,
// X3 = c f_S, X4 = c h_S, X5 = d g_W, X6 = d h_W; their unknowns are approximated by
// alpha (sum of the two stencil points minus the centre), and M equals K at K's positions:
//   b = K_B / (1 + alpha (f_B + g_B)),   c = K_S / (1 + alpha (f_S + h_S)),
//   d = K_W / (1 + alpha (g_W + h_W)),
//   e = K_P - b h_B - c g_S - d f_W + alpha (X1 + ... + X6),
//   f = (K_E - alpha (X1 + X3)) / e,   g = (K_N - alpha (X2 + X5)) / e,
//   h = (K_T - alpha (X4 + X6)) / e,
// every entry toward a node that is not an unknown being 0.  One iteration is r = rho - K phi,
// L v = r, U delta = v, phi += delta.
//
// The factorisation and both substitutions are recurrences along all three axes: node
// (i, j, k) needs its -x, -y, -z neighbours first (the +x, +y, +z ones going back), so the
// nodes of one hyperplane i + j + k = s depend only on the hyperplane before.  The interior is
// cut into tiles of at most SIP_TS^3 nodes, and the tiles of one hyperplane of tiles are one launch, a
// block each: a block loads its tile and the three faces next to it into LDS and walks the
// tile's (at most 3 SIP_TS - 2) hyperplanes there, one barrier apart.  A substitution on n^3 interior
// nodes takes 3 n / 16 - 2 launches instead of 3 n - 2 (one per hyperplane of nodes, 3 us
// each: 64^3 in FP64, 570 us per substitution; in tiles 10 launches of 13.5 us, of which the steps take 8).  What is left is the chain of
// the hyperplanes: an LDS read, three multiply-adds, a division and a barrier per step.
//
// Factors are stored per tile in hyperplane order (the nodes of a step are consecutive), in two
// arrays of four values: b, c, d, e for the forward substitution and f, g, h, 0 for the
// backward one.  Nodes that are not unknowns, and those of a tile beyond the interior, have
// b = c = d = f = g = h = 0 and e = 1: their value stays 0 without a test.
#include <hip/hip_runtime.h>

#include "cps_kernels.h"

namespace cps {

namespace {

constexpr int TS = SIP_TS, TN = SIP_TN, STEPS = SIP_STEPS;
// LDS tile (the tile and one face layer per axis): strides of j and k for which the nodes of a
// hyperplane, at s + (LY - 1) j + (LZ - 1) k, fall on different banks (17 j + 16 k modulo 32
// double or 64 float banks).  With strides 17 and 289 (16 j + 288 k) 32 lanes met on two banks:
// 18 us per launch at 64^3 in FP64, 13.5 us with these.
constexpr int LY = TS + 2, LZ = 337, LSIZE = LZ * (TS + 1);
static_assert(LZ >= LY * (TS + 1), "planes do not overlap");
constexpr int SIP_THREADS = 256;          // at least the nodes of the largest hyperplane (192)
// steps whose factors are loaded ahead: a step takes 0.16 us, a load up to about a microsecond
// (going back 14.2 us per launch with 4, 13.4 with 8)
constexpr int AHEAD = 8;

// The grid's tiles: TS nodes along every axis where they take at most FULL_MAX times the grid's nodes
// (their edges are constants of the kernels then); otherwise, on short axes, the same number of
// tiles with edges as equal as possible (18 interior nodes make two tiles of 9, 3 make one of 3), so
// that the factors never take much more memory than one set per node (5 x 200 x 200: 3.5 times).  Measured,
// FP32 / FP64 (ms a preconditioner apply, edges of TS against equal ones): 20^3 0.84 / 0.90 against 0.78 /
// 0.83; 130 x 20 x 20 2.03 / 2.17 against 1.90 / 2.05; 5 x 200 x 200 5.1 / 5.4 against 5.1 / 5.5.
constexpr double FULL_MAX = 1.5;
struct Tiles {
    int nt[3], ts[3];                     // tiles and nodes of a tile per axis
};
inline Tiles tiles_of(int nx, int ny, int nz)
{
    const int n[3] = {nx - 2, ny - 2, nz - 2};
    Tiles g;
    for (int d = 0; d < 3; ++d) {
        g.nt[d] = (n[d] + TS - 1) / TS;
        g.ts[d] = TS;
    }
    if ((double)TN * g.nt[0] * g.nt[1] * g.nt[2] > FULL_MAX * nx * ny * nz)
        for (int d = 0; d < 3; ++d) g.ts[d] = (n[d] + g.nt[d] - 1) / g.nt[d];
    return g;
}
inline bool full_tiles(const Tiles &g) { return g.ts[0] == TS && g.ts[1] == TS && g.ts[2] == TS; }
__host__ __device__ __forceinline__ int tile_nodes(const Tiles &g) { return g.ts[0] * g.ts[1] * g.ts[2]; }

constexpr SipOrder make_order(int ti, int tj, int tk)
{
    SipOrder o{};
    int q = 0;
    for (int s = 0; s < STEPS; ++s) {
        o.start[s] = q;
        for (int k = 0; k < tk; ++k)
            for (int j = 0; j < tj; ++j) {
                const int i = s - j - k;
                if (i < 0 || i >= ti) continue;
                const int n = i + TS * (j + TS * k);
                o.node[q] = (uint16_t)n;
                o.cell[q] = (uint16_t)(i + LY * j + LZ * k);
                o.pos[n] = (uint16_t)q;
                ++q;
            }
    }
    o.start[STEPS] = q;
    return o;
}
constexpr SipOrder FULL_ORDER = make_order(TS, TS, TS);
__device__ const SipOrder full_order = FULL_ORDER;

__device__ __forceinline__ bool unk(int8_t t) { return t == 1 || t == 2; }

// a hyperplane of tiles: blocks over (tile j, tile k), tile i = s - tile j - tile k
struct TilePlane {
    int s, klo;
};

struct Tile {
    int i, j, k;                          // tile indices
    int o[3];                             // first node
    size_t base;                          // first entry of its factors
    bool ok;
};
__device__ __forceinline__ Tile tile_of(const Tiles &g, const TilePlane &p)
{
    Tile t;
    t.j = (int)blockIdx.x;
    t.k = p.klo + (int)blockIdx.y;
    t.i = p.s - t.j - t.k;
    t.ok = t.i >= 0 && t.i < g.nt[0];
    t.o[0] = 1 + g.ts[0] * t.i;
    t.o[1] = 1 + g.ts[1] * t.j;
    t.o[2] = 1 + g.ts[2] * t.k;
    t.base = ((size_t)t.i + (size_t)g.nt[0] * (t.j + (size_t)g.nt[1] * t.k)) * tile_nodes(g);
    return t;
}

template <typename T>
struct alignas(4 * sizeof(T)) Four {
    T v[4];
};

// Factors of one hyperplane of tiles.  f, g, h of the tile and of the three faces below it
// live in LDS (index i + LY j + LZ k, 0 being the face).
__global__ void __launch_bounds__(SIP_THREADS) k_sip_factor(int nx, int ny, int nz, Tiles g, TilePlane p,
                                                            const SipOrder *__restrict__ order, Coef<double> cf,
                                                            const int8_t *__restrict__ type,
                                                            const int *__restrict__ irr_map,
                                                            const double *__restrict__ k7, double alpha,
                                                            Four<double> *__restrict__ L, Four<double> *__restrict__ U,
                                                            Four<float> *__restrict__ L32, Four<float> *__restrict__ U32)
{
    __shared__ double sf[3][LSIZE];
    const Tile t = tile_of(g, p);
    if (!t.ok) return;
    const int tid = (int)threadIdx.x;
    // the faces: the last layer of the tiles before, zero at the walls
    const int fa = tid % TS, fb = tid / TS;
    const size_t tn = tile_nodes(g), back[3] = {tn, tn * g.nt[0], tn * g.nt[0] * g.nt[1]};
    const int at[3] = {LY * (fa + 1) + LZ * (fb + 1), fa + 1 + LZ * (fb + 1), fa + 1 + LY * (fb + 1)};
    const int nb[3] = {g.ts[0] - 1 + TS * (fa + TS * fb), fa + TS * (g.ts[1] - 1 + TS * fb),
                       fa + TS * (fb + TS * (g.ts[2] - 1))};
    const int tix[3] = {t.i, t.j, t.k};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        Four<double> u{};
        if (tix[d] > 0 && fa < g.ts[d == 0 ? 1 : 0] && fb < g.ts[d == 2 ? 1 : 2]) u = U[t.base - back[d] + order->pos[nb[d]]];
#pragma unroll
        for (int q = 0; q < 3; ++q) sf[q][at[d]] = u.v[q];
    }
    __syncthreads();
    const size_t sy = nx, sz = (size_t)nx * ny;
    for (int s = 0; s < STEPS; ++s) {
        const int q = order->start[s] + tid;
        if (q < order->start[s + 1]) {
            const int n = order->node[q], li = n % TS, lj = (n / TS) % TS, lk = n / (TS * TS);
            const int i = t.o[0] + li, j = t.o[1] + lj, k = t.o[2] + lk;
            const int c0 = (li + 1) + LY * (lj + 1) + LZ * (lk + 1);
            double lo[4] = {0.0, 0.0, 0.0, 1.0}, up[4] = {0.0, 0.0, 0.0, 0.0};
            const bool in = i <= nx - 2 && j <= ny - 2 && k <= nz - 2;
            const size_t e = in ? (size_t)i + sy * j + sz * k : 0;
            const int8_t ty = in ? type[e] : (int8_t)0;
            if (unk(ty)) {
                const bool xe = unk(type[e + 1]), yn = unk(type[e + sy]), zt = unk(type[e + sz]);
                double co[7];
                if (ty == 2) {
                    const double *r = k7 + 7 * (size_t)irr_map[e];
#pragma unroll
                    for (int w = 0; w < 7; ++w) co[w] = r[w];
                } else {
                    const double *cx = cf.c[0] + 8 * i, *cy = cf.c[1] + 8 * j, *cz = cf.c[2] + 8 * k;
                    co[0] = (cx[6] + cy[6]) + cz[6];
                    co[1] = unk(type[e - 1]) ? cx[5] : 0.0;
                    co[2] = xe ? cx[7] : 0.0;
                    co[3] = unk(type[e - sy]) ? cy[5] : 0.0;
                    co[4] = yn ? cy[7] : 0.0;
                    co[5] = unk(type[e - sz]) ? cz[5] : 0.0;
                    co[6] = zt ? cz[7] : 0.0;
                }
                // f, g, h of the -z, -y, -x neighbours (zero at nodes that are not unknowns)
                const int cB = c0 - LZ, cS = c0 - LY, cW = c0 - 1;
                const double fB = sf[0][cB], gB = sf[1][cB], hB = sf[2][cB];
                const double fS = sf[0][cS], gS = sf[1][cS], hS = sf[2][cS];
                const double fW = sf[0][cW], gW = sf[1][cW], hW = sf[2][cW];
                const double b = co[5] / (1.0 + alpha * (fB + gB));
                const double c = co[3] / (1.0 + alpha * (fS + hS));
                const double d = co[1] / (1.0 + alpha * (gW + hW));
                const double X1 = b * fB, X2 = b * gB, X3 = c * fS, X4 = c * hS, X5 = d * gW, X6 = d * hW;
                const double ee = co[0] - b * hB - c * gS - d * fW + alpha * (X1 + X2 + X3 + X4 + X5 + X6);
                lo[0] = b;
                lo[1] = c;
                lo[2] = d;
                lo[3] = ee;
                up[0] = xe ? (co[2] - alpha * (X1 + X3)) / ee : 0.0;
                up[1] = yn ? (co[4] - alpha * (X2 + X5)) / ee : 0.0;
                up[2] = zt ? (co[6] - alpha * (X4 + X6)) / ee : 0.0;
            }
#pragma unroll
            for (int w = 0; w < 3; ++w) sf[w][c0] = up[w];
            Four<double> l4, u4;
            Four<float> l4f, u4f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                l4.v[w] = lo[w];
                u4.v[w] = up[w];
                l4f.v[w] = (float)lo[w];
                u4f.v[w] = (float)up[w];
            }
            L[t.base + q] = l4;
            U[t.base + q] = u4;
            L32[t.base + q] = l4f;
            U32[t.base + q] = u4f;
        }
        __syncthreads();
    }
}

// One hyperplane of tiles of a substitution.
//   FWD  L v = r:      v = (r - b v_B - c v_S - d v_W) / e
//   else U delta = v:  delta = v - (f delta_E + g delta_N + h delta_T), delta over v, and
//                      phi = delta (first iteration) or phi += delta
// The tile and the face layer it depends on (below it going forward, above it going back) are
// in LDS; values are replaced in place, hyperplane by hyperplane.  FULL: tiles of TS nodes along every
// axis, with their edges and order as constants (64^3 FP32: 2.07 ms an apply, 2.29 with edges
// and order read).
template <typename T, bool FWD, bool FULL>
__global__ void __launch_bounds__(SIP_THREADS) k_sip_sub(int nx, int ny, int nz, Tiles g, TilePlane p,
                                                         const SipOrder *__restrict__ tile_order,
                                                         const Four<T> *__restrict__ F, const T *__restrict__ r, T *v,
                                                         T *__restrict__ phi, int first, const DevState *st)
{
    __shared__ T w[LSIZE];
    __shared__ uint4 cells[TN / 8];       // the order's cells, staged with the tile
    if (FULL) g.ts[0] = g.ts[1] = g.ts[2] = TS;
    const SipOrder *order = FULL ? &full_order : tile_order;
    const Tile t = tile_of(g, p);
    if (!t.ok) return;
    const int done = st ? st->done : 0;   // used at the end: nothing waits for it
    const int tid = (int)threadIdx.x;
    const size_t sy = nx, sz = (size_t)nx * ny;
    constexpr int SH = FWD ? 1 : 0;       // the face layer is LDS layer 0 (forward) or TS (back)
    const T *src = FWD ? r : v;
    // the hyperplanes' first positions, one per lane (read by step)
    const int starts = order->start[min(tid & 63, STEPS)];
    auto start_of = [&](int s) { return __builtin_amdgcn_readlane(starts, FWD ? s : STEPS - 1 - s); };
    auto count_of = [&](int s) { return __builtin_amdgcn_readlane(starts, FWD ? s + 1 : STEPS - s) - start_of(s); };
    const uint4 *cell_src = reinterpret_cast<const uint4 *>(order->cell);
    const uint4 cl[2] = {cell_src[tid], cell_src[tid + SIP_THREADS]};
    static_assert(TN == 16 * SIP_THREADS, "two loads per thread hold the cells");
    // factors of the first steps
    const Four<T> *Ft = F + t.base;
    const int tlast = FULL ? TN - 1 : tile_nodes(g) - 1;
    Four<T> fr[AHEAD];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) fr[s] = Ft[min(start_of(s) + tid, tlast)];
    // the tile and its faces (walls hold 0; nodes beyond the interior are taken as 0): all loads
    // are issued before the first value is used, from clamped addresses (node 0 is a wall)
    constexpr int NU = TN / SIP_THREADS;
    T tv[NU], fv[3];
    bool tin[NU], fin[3];
    auto own = [&](int n) { return FULL || ((n % TS < g.ts[0]) & ((n / TS) % TS < g.ts[1]) & (n / (TS * TS) < g.ts[2])); };
    int fat[3];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int n = tid + SIP_THREADS * u, li = n % TS, lj = (n / TS) % TS, lk = n / (TS * TS);
        const int i = t.o[0] + li, j = t.o[1] + lj, k = t.o[2] + lk;
        if constexpr (FULL) tin[u] = i <= nx - 2 && j <= ny - 2 && k <= nz - 2;
        else tin[u] = own(n) & (i <= nx - 2) & (j <= ny - 2) & (k <= nz - 2);
        tv[u] = src[tin[u] ? (size_t)i + sy * j + sz * k : 0];
    }
    const int fa = tid % TS, fb = tid / TS;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int off = FWD ? -1 : g.ts[d], at = FWD ? 0 : g.ts[d];
        const int l[3] = {d == 0 ? off : fa, d == 1 ? off : (d == 0 ? fa : fb), d == 2 ? off : fb};
        const int c[3] = {d == 0 ? at : fa + SH, d == 1 ? at : (d == 0 ? fa : fb) + SH, d == 2 ? at : fb + SH};
        const int i = t.o[0] + l[0], j = t.o[1] + l[1], k = t.o[2] + l[2];
        fin[d] = i >= 1 && j >= 1 && k >= 1 && i <= nx - 2 && j <= ny - 2 && k <= nz - 2;
        if constexpr (!FULL) fin[d] = fin[d] & (fa < g.ts[d == 0 ? 1 : 0]) & (fb < g.ts[d == 2 ? 1 : 2]);
        fv[d] = v[fin[d] ? (size_t)i + sy * j + sz * k : 0];
        fat[d] = c[0] + LY * c[1] + LZ * c[2];
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int n = tid + SIP_THREADS * u, li = n % TS, lj = (n / TS) % TS, lk = n / (TS * TS);
        if (own(n)) w[(li + SH) + LY * (lj + SH) + LZ * (lk + SH)] = tin[u] ? tv[u] : T(0);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) w[fat[d]] = fin[d] ? fv[d] : T(0);
    cells[tid] = cl[0];
    cells[tid + SIP_THREADS] = cl[1];
    __syncthreads();
    const uint16_t *cell = reinterpret_cast<const uint16_t *>(cells);
    int n_next = cell[min(start_of(0) + tid, TN - 1)];
#pragma unroll
    for (int s0 = 0; s0 < STEPS; s0 += AHEAD) {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            const int s = s0 + a;
            if (s >= STEPS) break;
            const Four<T> f = fr[a];
            const int n = n_next, cnt = count_of(s);
            if (s + AHEAD < STEPS) fr[a] = Ft[min(start_of(s + AHEAD) + tid, tlast)];
            if (s + 1 < STEPS) n_next = cell[min(start_of(s + 1) + tid, TN - 1)];
            if (tid < cnt) {
                const int c0 = n + SH * (1 + LY + LZ);
                if (FWD) w[c0] = (w[c0] - f.v[0] * w[c0 - LZ] - f.v[1] * w[c0 - LY] - f.v[2] * w[c0 - 1]) / f.v[3];
                else w[c0] = w[c0] - (f.v[0] * w[c0 + 1] + f.v[1] * w[c0 + LY] + f.v[2] * w[c0 + LZ]);
            }
            __syncthreads();
        }
    }
    if (done) return;
    T pv[NU];
    if (!FWD)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int n = tid + SIP_THREADS * u, li = n % TS, lj = (n / TS) % TS, lk = n / (TS * TS);
            pv[u] = first ? T(0) : phi[tin[u] ? (size_t)(t.o[0] + li) + sy * (t.o[1] + lj) + sz * (t.o[2] + lk) : 0];
        }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int n = tid + SIP_THREADS * u, li = n % TS, lj = (n / TS) % TS, lk = n / (TS * TS);
        if (!tin[u]) continue;
        const size_t e = (size_t)(t.o[0] + li) + sy * (t.o[1] + lj) + sz * (t.o[2] + lk);
        const T val = w[(li + SH) + LY * (lj + SH) + LZ * (lk + SH)];
        v[e] = val;
        if (!FWD) phi[e] = first ? val : pv[u] + val;
    }
}

// launch shape of a hyperplane of tiles: blocks over tile j, and the tile k that reach it
inline bool plane_launch(const Tiles &g, int s, TilePlane &p, dim3 &grid)
{
    const int klo = std::max(0, s - (g.nt[0] - 1) - (g.nt[1] - 1)), khi = std::min(g.nt[2] - 1, s);
    if (khi < klo) return false;
    p.s = s;
    p.klo = klo;
    grid = dim3((unsigned)g.nt[1], (unsigned)(khi - klo + 1));
    return true;
}

inline int tile_planes(const Tiles &g) { return g.nt[0] + g.nt[1] + g.nt[2] - 2; }

}  // namespace

SipOrder sip_order(int nx, int ny, int nz)
{
    const Tiles g = tiles_of(nx, ny, nz);
    return make_order(g.ts[0], g.ts[1], g.ts[2]);
}

size_t sip_factor_nodes(int nx, int ny, int nz)
{
    const Tiles g = tiles_of(nx, ny, nz);
    return (size_t)g.nt[0] * g.nt[1] * g.nt[2] * tile_nodes(g);
}

void launch_sip_factor(hipStream_t st, int nx, int ny, int nz, const SipOrder *order, const Coef<double> &cf,
                       const int8_t *type, const int *irr_map, const double *k7, double alpha, double *F, float *F32)
{
    const size_t nf = sip_factor_nodes(nx, ny, nz);
    const Tiles g = tiles_of(nx, ny, nz);
    Four<double> *L = reinterpret_cast<Four<double> *>(F);
    Four<float> *L32 = reinterpret_cast<Four<float> *>(F32);
    for (int s = 0; s < tile_planes(g); ++s) {
        TilePlane p;
        dim3 grid;
        if (plane_launch(g, s, p, grid))
            k_sip_factor<<<grid, SIP_THREADS, 0, st>>>(nx, ny, nz, g, p, order, cf, type, irr_map, k7, alpha, L, L + nf, L32,
                                                       L32 + nf);
    }
}

template <typename T>
void launch_sip_iteration(hipStream_t st, int nx, int ny, int nz, const SipOrder *order, const T *F, const T *r, T *v,
                          T *phi, int first, const DevState *dst)
{
    const Four<T> *L = reinterpret_cast<const Four<T> *>(F), *U = L + sip_factor_nodes(nx, ny, nz);
    const Tiles g = tiles_of(nx, ny, nz);
    const int np = tile_planes(g);
    const auto fwd = full_tiles(g) ? &k_sip_sub<T, true, true> : &k_sip_sub<T, true, false>;
    const auto back = full_tiles(g) ? &k_sip_sub<T, false, true> : &k_sip_sub<T, false, false>;
    for (int s = 0; s < np; ++s) {
        TilePlane p;
        dim3 grid;
        if (plane_launch(g, s, p, grid))
            fwd<<<grid, SIP_THREADS, 0, st>>>(nx, ny, nz, g, p, order, L, r, v, nullptr, 0, dst);
    }
    for (int s = np - 1; s >= 0; --s) {
        TilePlane p;
        dim3 grid;
        if (plane_launch(g, s, p, grid))
            back<<<grid, SIP_THREADS, 0, st>>>(nx, ny, nz, g, p, order, U, nullptr, v, phi, first, dst);
    }
}

template void launch_sip_iteration<double>(hipStream_t, int, int, int, const SipOrder *, const double *, const double *,
                                           double *, double *, int, const DevState *);
template void launch_sip_iteration<float>(hipStream_t, int, int, int, const SipOrder *, const float *, const float *,
                                          float *, float *, int, const DevState *);

}  // namespace cps
