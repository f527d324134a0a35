// multigrid.hip -- grid transfers of the multigrid preconditioner for K.
//
// The paper preconditions BiCGSTAB with the second-order operator K (Sec. 3.3) applied
// approximately by an inner solver, and allows other inner solvers than its own.  The
// multigrid inner solver is one V-cycle on a hierarchy of grids: a coarser grid keeps, along
// every axis, the even-indexed points and the last one, and carries its own K built from the
// level set at its nodes.  Prolongation P is the tensor product of 1D linear interpolation
// in the physical coordinate; restriction is P^T with every coarse row divided by its sum.
// Both act on unknown nodes only: every other node holds 0 on every level; the coarse
// correction is added at the regular unknown nodes (not at the irregular ones).
//
// 1D tables per axis (built on the host from the coordinates):
//   prolongation  for each fine index i, whose left coarse index is a = min(i / 2, nc - 2):
//                 the weight w[i] of coarse node a + 1 (fine value = (1 - w) e[a] +
//                 w e[a + 1]); the weights carry 4 zeros of padding
//   restriction   for each interior coarse index I (fine point 2I): the weights rw[3I + q]
//                 of fine points 2I - 1 + q, q = 0 .. 2, already divided by the row sum
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "cps_kernels.h"

namespace cps {

namespace {

__device__ __forceinline__ bool unknown(int8_t t) { return t == 1 || t == 2; }

template <typename T>
struct MgVec4;
template <>
struct MgVec4<float> {
    typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct MgVec4<double> {
    typedef double type __attribute__((ext_vector_type(4), aligned(8)));
};

// Coarse rho(I, J, K) = sum over the 3 x 3 x 3 fine nodes (2I - 1 .. 2I + 1, ...) of
// rwx rwy rwz r at the unknown coarse nodes, 0 at the other interior nodes (the walls of rc
// are never written and stay 0).  Block 64 x 4: lane l takes the interior coarse nodes
// I0 = 1 + 128 blockIdx.x + 2 l and I0 + 1 of row J = 1 + 4 blockIdx.y + wavefront, plane
// K = 1 + blockIdx.z; it reads fine nodes 2 I0 - 1 .. 2 I0 + 2 of each of the nine fine
// rows as a 4-vector, and node 2 I0 + 3 from the next lane.  Every load is issued whatever
// the node types.
// With a first step F (F.x1 non-null) it also writes the coarse level's first Chebyshev
// step from zero, x1 = c2 rho / diag K, at its unknown nodes.
template <typename T>
__global__ void __launch_bounds__(256) k_mg_restrict(int ncx, int ncy, int nfx, int nfy, MgAxis<T> ax, MgAxis<T> ay,
                                                     MgAxis<T> az, const T *__restrict__ r, T *__restrict__ rc,
                                                     MgFirst<T> F)
{
    using V = typename MgVec4<T>::type;
    const int I0 = 1 + (int)(blockIdx.x * 128 + 2 * threadIdx.x), J = 1 + (int)(blockIdx.y * 4 + threadIdx.y);
    const int K = 1 + (int)blockIdx.z;
    if (I0 > ncx - 2 || J > ncy - 2) return;
    const bool two = I0 + 1 <= ncx - 2;
    const int I1 = two ? I0 + 1 : I0;
    T w0[3], w1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        w0[a] = ax.rw[3 * I0 + a];
        w1[a] = ax.rw[3 * I1 + a];
    }
    const size_t ec = (size_t)I0 + (size_t)ncx * (J + (size_t)ncy * K);
    const T dg0 = F.diag[ec], dg1 = two ? F.diag[ec + 1] : T(0);
    const bool unk0 = dg0 != T(0), unk1 = dg1 != T(0);
    const size_t fplane = (size_t)nfx * nfy;
    const int f0 = 2 * I0 - 1;                      // first fine node of the lane
    const int f4 = min(f0 + 4, nfx - 1);            // fifth node (I0 + 1's last), in the row
    // the fifth node is the next lane's first one, taken by a shuffle unless that lane has no
    // coarse node (then the lane loads it)
    const bool self4 = threadIdx.x == 63 || I0 + 2 > ncx - 2;
    T acc0 = T(0), acc1 = T(0);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const T wz = az.rw[3 * K + c];
        const size_t kz = (size_t)(2 * K - 1 + c) * fplane;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const T wyz = wz * ay.rw[3 * J + b];
            const T *row = r + kz + (size_t)(2 * J - 1 + b) * nfx;
            const V v = *reinterpret_cast<const V *>(row + f0);
            T v4 = __shfl_down(v.x, 1, 64);
            if (self4) v4 = row[f4];
            acc0 += wyz * (w0[0] * v.x + w0[1] * v.y + w0[2] * v.z);
            acc1 += wyz * (w1[0] * v.z + w1[1] * v.w + w1[2] * v4);
        }
    }
    rc[ec] = unk0 ? acc0 : T(0);
    if (two) rc[ec + 1] = unk1 ? acc1 : T(0);
    if (F.x1) {
        if (unk0) F.x1[ec] = F.c2 * acc0 / dg0;
        if (unk1) F.x1[ec + 1] = F.c2 * acc1 / dg1;
    }
}

// A wave-uniform value moved to a scalar register.
__device__ __forceinline__ float wave_uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double wave_uniform(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// rho - K x at a regular node from its seven x values (centre c, then the -x, +x, -y, +y,
// -z, +z neighbours) and the 1D tables of its three indices (Eq. 2ndorder_coef).
template <typename T>
__device__ __forceinline__ T mg_reg_resid(T rh, T c, T w, T e, T s, T n, T m, T u, T kax, T kbx, T kcx, T kay,
                                          T kby, T kcy, T za, T zb, T zc)
{
    const T kd = kbx + kby + zb;
    return rh - (kd * c + kax * w + kcx * e + kay * s + kcy * n + za * m + zc * u);
}

// Residual and restriction in one pass on the problem's grid: rc = R (rho - K x) at the
// unknown coarse nodes, 0 at the other interior ones (the sums of k_mg_restrict), with no fine
// residual stored.  A block owns RR_ROWS coarse rows of a 128-node coarse segment bs and the
// coarse planes K0 .. K1 - 1 of a chunk, and has a wavefront more than rows: wavefront w forms
// the residual of fine rows 2J - 1 and 2J, J = J0 + w, so that no wavefront forms a row twice.
// Both belong to coarse row J; row 2J - 1 is also the last of coarse row J - 1, whose wavefront
// gets that share, summed over the three fine planes of a coarse plane, through LDS (the
// wavefront beyond the block's rows works for that share alone).
// Lane l takes coarse nodes I0 = 1 + 128 bs + 2 l and I0 + 1, whose fine points are
// f0 = 2 I0 - 1 .. f0 + 4: it forms the residual at f0 .. f0 + 3 (the four-node layout of the
// vectorised sweeps) and takes the one at f0 + 4 from the next lane; the last lane forms its own
// fifth node when its segment owns I0 + 1 and f0 + 4 is interior (FIFTH).  One load per row and
// plane brings both ends of a segment what they need beyond it: nodes f0 + 4 and f0 + 5 in lane 63,
// f0 - 1 in lane 0.
// The wavefronts march over the fine planes 2 K0 - 1 .. 2 K1 - 1, x of the planes below and above
// carried in registers; coarse plane K is complete, and stored, after fine plane 2K + 1.  The
// first fine plane of a chunk is formed by both chunks.
// Irregular and solid fine nodes (skip bits) take their residual from ri, which holds it
// at the irregular nodes (the irregular rows of the residual kernel, run before) and 0 at
// the solid ones; walls give 0.  With a first step F (F.x1 non-null) the coarse level's first Chebyshev
// step from zero is written too, as k_mg_restrict does.
// Where a fine row has at most 128 interior nodes (HALF), a wavefront takes two coarse rows, half of
// its lanes each: no lane idles, and a block's 15 rows leave room for chunks of one plane (128^3
// FP32 11.3 us against 14.8, 12.3 with chunks of two; 98^3 FP64 9.8 against 13.2).
// Bound by its loads (instructions and round trips per plane).  Against one coarse row per
// wavefront with its three fine rows, four wavefronts a block (us): 512^3 FP32 363 against 505; 256^3
// FP32 40.5 against 49.6; 200^3 FP32 24 against 31.  Seven rows: with 3 /
// 4 / 8 rows 256^3 FP32 takes 44 / 61 / 42 and FP64 104 / 98 / 115 against 40.5 and 88 (eight
// wavefronts fill a CU's registers evenly).  Loading a plane ahead is slower (48 at 256^3: the
// registers cost a quarter of the wavefronts).
// Loads through a buffer resource based at a wave-uniform address (one plane of an
// array): the 32-bit byte offset of each lane goes in a vector register and the base in
// scalar registers, so an address costs no 64-bit vector arithmetic (this kernel issues
// about twenty loads per plane step, and its throughput is bound by instruction issue).
typedef uint32_t MgU4 __attribute__((ext_vector_type(4)));
struct MgF4 {
    float v[4];
};
struct MgD2 {
    double v[2];
};
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *base)
{
    // raw buffer (stride 0), range 4 GiB from the base, 32-bit data format (CDNA)
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, -1, 0x00020000);
}
template <typename T>
__device__ __forceinline__ typename MgVec4<T>::type bload4(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <>
__device__ __forceinline__ MgVec4<float>::type bload4<float>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    const MgF4 f = __builtin_bit_cast(MgF4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    return MgVec4<float>::type{f.v[0], f.v[1], f.v[2], f.v[3]};
}
template <>
__device__ __forceinline__ MgVec4<double>::type bload4<double>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    const MgD2 a = __builtin_bit_cast(MgD2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    const MgD2 b = __builtin_bit_cast(MgD2, __builtin_amdgcn_raw_buffer_load_b128(r, off + 16, 0, 0));
    return MgVec4<double>::type{a.v[0], a.v[1], b.v[0], b.v[1]};
}
template <typename T>
__device__ __forceinline__ T bload1(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <>
__device__ __forceinline__ float bload1<float>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
template <>
__device__ __forceinline__ double bload1<double>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <typename T>
struct MgPair {
    T a, b;
};
template <typename T>
__device__ __forceinline__ MgPair<T> bload2(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <>
__device__ __forceinline__ MgPair<float> bload2<float>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(MgPair<float>, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <>
__device__ __forceinline__ MgPair<double> bload2<double>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(MgPair<double>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ uint64_t bload_u64(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}

// coarse rows of a block
constexpr int RR_ROWS = 7;

template <typename T, bool FIFTH, bool HALF>
__global__ void __launch_bounds__(64 * (RR_ROWS + 1)) k_mg_resid_restrict(Geom g, Tiling tl, Coef<T> cf,
                                                           const uint32_t *__restrict__ skip,
                                                           const T *__restrict__ x, const T *__restrict__ rho,
                                                           const T *__restrict__ ri, int ncx, int ncy, int ncz,
                                                           MgAxis<T> ax, MgAxis<T> ay, MgAxis<T> az,
                                                           T *__restrict__ rc, MgFirst<T> F, const DevState *st)
{
    using V = typename MgVec4<T>::type;
    constexpr int LANES = HALF ? 32 : 64, SLOTS = 64 / LANES * (RR_ROWS + 1), ROWS = SLOTS - 1;
    __shared__ T sh[2][SLOTS][2][LANES];                      // row 2J - 1's share of coarse row J - 1
    auto uni = [](T v) { return HALF ? v : wave_uniform(v); };   // a value of the coarse row
    if (st && st->done) return;
    int bs, by, bz;
    if (!tile_of_block(tl, (int)blockIdx.x, bs, by, bz)) return;
    const int lane = (int)threadIdx.x % LANES, wv = ((int)threadIdx.x + 64 * (int)threadIdx.y) / LANES;
    const int J = 1 + by * ROWS + wv;                          // the lanes' coarse row (up to ncy - 2 + ROWS)
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const size_t plane = (size_t)nx * ny, wplane = (size_t)ny * g.W;
    const int I0 = 1 + 128 * bs + 2 * lane;
    const bool own0 = I0 <= ncx - 2, own1 = I0 + 1 <= ncx - 2;
    const int f0 = 2 * I0 - 1;
    const int nv = min(4, nx - 1 - f0);                       // interior fine nodes of the lane
    // the lane's loads start at node ic: f0, or the wall node for lanes past the row end.
    // Values past the lane's valid nodes are never used: their residuals are zeroed, and
    // the +x neighbour of the last interior node is the wall node (0 in every vector).
    const int ic = min(f0, nx - 1);
    const bool need5 = FIFTH && lane == LANES - 1 && own1 && f0 + 4 <= nx - 2;
    const bool needl = FIFTH && lane == 0 && bs > 0;          // node f0 - 1 is interior
    const bool edge = need5 || needl;
    const uint32_t eoff = (uint32_t)((need5 ? 4 : -1) * (int)sizeof(T));   // from node ic to the edge pair
    // the skip bits that matter: the lane's interior nodes, and the fifth node where formed
    const uint32_t smask = ((1u << max(nv, 0)) - 1u) | (need5 ? 0x10u : 0u);
    T w0[3], w1[3];
    {
        const int a0 = own0 ? I0 : 1, a1 = own1 ? I0 + 1 : a0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            w0[a] = ax.rw[3 * a0 + a];
            w1[a] = ax.rw[3 * a1 + a];
        }
    }
    T kax[5], kbx[5], kcx[5];
    {
        const T *x5 = cf.xs + (size_t)5 * cf.xp + ic, *x6 = x5 + cf.xp, *x7 = x6 + cf.xp;
        const V va = *reinterpret_cast<const V *>(x5), vb = *reinterpret_cast<const V *>(x6),
                vc = *reinterpret_cast<const V *>(x7);
        const T a[5] = {va.x, va.y, va.z, va.w, x5[4]}, bb[5] = {vb.x, vb.y, vb.z, vb.w, x6[4]},
                c[5] = {vc.x, vc.y, vc.z, vc.w, x7[4]};
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            kax[u] = a[u];
            kbx[u] = bb[u];
            kcx[u] = c[u];
        }
    }
    // in-plane byte offsets of node ic on x rows 2J - 2 .. 2J + 1 (clamped to the wall row, where
    // x is 0); the residual rows 2J - 1 and 2J are x rows 1 and 2, those past the last interior
    // row zeroed; ow: byte offsets of their skip words
    uint32_t ox[4], ow[2];
#pragma unroll
    for (int c = 0; c < 4; ++c) ox[c] = (uint32_t)((ic + nx * min(2 * J - 2 + c, ny - 1)) * sizeof(T));
    bool rok[2];
    T kay[2], kby[2], kcy[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int j = 2 * J - 1 + b;
        rok[b] = j <= ny - 2;
        const int jc = min(j, ny - 1);
        ow[b] = (uint32_t)((jc * g.W + (ic >> 5)) * sizeof(uint32_t));
        kay[b] = uni(cf.c[1][8 * jc + 5]);
        kby[b] = uni(cf.c[1][8 * jc + 6]);
        kcy[b] = uni(cf.c[1][8 * jc + 7]);
    }
    // the y weights of rows 2J - 1 and 2J in coarse row J, and of row 2J - 1 in coarse row J - 1
    const bool jok = wv < ROWS && J <= ncy - 2;             // the wavefront stores coarse row J
    const int Jc = min(J, ncy - 2), Jp = min(J - 1, ncy - 2);
    const T wy0 = uni(ay.rw[3 * Jc]), wy1 = uni(ay.rw[3 * Jc + 1]);
    const T wyp = (wv > 0 && J - 1 <= ncy - 2) ? uni(ay.rw[3 * Jp + 2]) : T(0);

    const int K0 = 1 + bz * tl.TZ, K1 = min(K0 + tl.TZ, ncz - 1);
    const int p0 = 2 * K0 - 1, p1 = 2 * K1 - 1;
    // x of the residual rows at the plane below (m) and at the current one (c); their edge pairs
    V xm[2], xc[2];
    MgPair<T> em[2], ec[2];
    {
        const __amdgpu_buffer_rsrc_t xb = plane_rsrc(x + (size_t)(p0 - 1) * plane), x0 = plane_rsrc(x + (size_t)p0 * plane);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            xm[b] = bload4<T>(xb, ox[b + 1]);
            xc[b] = bload4<T>(x0, ox[b + 1]);
            em[b] = edge ? bload2<T>(xb, ox[b + 1] + eoff) : MgPair<T>{T(0), T(0)};
            ec[b] = edge ? bload2<T>(x0, ox[b + 1] + eoff) : MgPair<T>{T(0), T(0)};
        }
    }
    // the coarse plane being summed: the diagonals of its nodes (0 where not an unknown),
    // loaded when the plane opens and used when it is stored two fine planes later; prv: the
    // share of coarse row J - 1
    T acc[2] = {T(0), T(0)}, prv[2] = {T(0), T(0)}, dg[2] = {T(0), T(0)};
    const size_t erow = (size_t)(own0 ? I0 : 1) + (size_t)ncx * Jc, cplane = (size_t)ncx * ncy;
    auto open = [&](int K) {
        const size_t e = erow + cplane * K;
        acc[0] = acc[1] = prv[0] = prv[1] = T(0);
        dg[0] = (own0 && jok) ? F.diag[e] : T(0);
        dg[1] = (own1 && jok) ? F.diag[e + 1] : T(0);
    };
    auto emit = [&](int K) {
        sh[K & 1][wv][0][lane] = prv[0];
        sh[K & 1][wv][1][lane] = prv[1];
        __syncthreads();
        if (!jok) return;
        const T a0 = acc[0] + sh[K & 1][wv + 1][0][lane], a1 = acc[1] + sh[K & 1][wv + 1][1][lane];
        const size_t e = erow + cplane * K;
        if (own0) rc[e] = dg[0] != T(0) ? a0 : T(0);
        if (own1) rc[e + 1] = dg[1] != T(0) ? a1 : T(0);
        if (F.x1) {
            if (dg[0] != T(0)) F.x1[e] = F.c2 * a0 / dg[0];
            if (dg[1] != T(0)) F.x1[e + 1] = F.c2 * a1 / dg[1];
        }
    };
    // coarse plane K += its z weight q times the fine plane's rows, restricted in y
    auto add_plane = [&](int K, int q, const T (&xr)[2][2]) {
        const T wz = wave_uniform(az.rw[3 * K + q]);
        const T c0 = wz * wy0, c1 = wz * wy1, cp = wz * wyp;
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            acc[o] += c0 * xr[0][o] + c1 * xr[1][o];
            prv[o] += cp * xr[0][o];
        }
    };
    // skip bits of nodes ic .. ic + 4 on the residual rows of plane q (words read in pairs;
    // the array carries two words of padding), loaded one plane ahead
    auto skip_bits = [&](int q, int b) -> uint32_t {
        return (uint32_t)(bload_u64(plane_rsrc(skip + (size_t)q * wplane), ow[b]) >> (ic & 31)) & smask;
    };
    uint32_t skn[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) skn[b] = skip_bits(p0, b);
    for (int p = p0; p <= p1; ++p) {
        const bool pv = p <= nz - 2;                          // fine plane p is interior
        const size_t kp = (size_t)p * plane;
        const __amdgpu_buffer_rsrc_t xk = plane_rsrc(x + kp), xn = plane_rsrc(x + (size_t)min(p + 1, nz - 1) * plane);
        const __amdgpu_buffer_rsrc_t rk = plane_rsrc(rho + kp), rik = plane_rsrc(ri + kp);
        V xp[2], rh[2], ri4[2];
        MgPair<T> ep[2];
        uint32_t sk[2];
        T h5[2], ri5[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const uint32_t o = ox[b + 1];
            sk[b] = skn[b];
            skn[b] = skip_bits(min(p + 1, nz - 1), b);
            xp[b] = bload4<T>(xn, o);
            rh[b] = bload4<T>(rk, o);
            // the residual at the lane's solid and irregular nodes (issued with the other loads)
            if (sk[b]) ri4[b] = bload4<T>(rik, o);
            else ri4[b] = V{T(0), T(0), T(0), T(0)};
            ri5[b] = (FIFTH && ((sk[b] >> 4) & 1u)) ? bload1<T>(rik, o + 4 * sizeof(T)) : T(0);
            ep[b] = edge ? bload2<T>(xn, o + eoff) : MgPair<T>{T(0), T(0)};
            h5[b] = need5 ? bload1<T>(rk, o + 4 * sizeof(T)) : T(0);
        }
        // the outer y neighbours: x rows 0 and 3
        const V ylo = bload4<T>(xk, ox[0]), yhi = bload4<T>(xk, ox[3]);
        const T ylo5 = need5 ? bload1<T>(xk, ox[0] + 4 * sizeof(T)) : T(0);
        const T yhi5 = need5 ? bload1<T>(xk, ox[3] + 4 * sizeof(T)) : T(0);
        const T *cz = cf.c[2] + 8 * p;
        const T za = wave_uniform(cz[5]), zb = wave_uniform(cz[6]), zc = wave_uniform(cz[7]);
        T xr[2][2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const V &s4 = b == 0 ? ylo : xc[0];
            const V &n4 = b == 0 ? xc[1] : yhi;
            const T cv[5] = {xc[b].x, xc[b].y, xc[b].z, xc[b].w, ec[b].a};
            const T sv[5] = {s4.x, s4.y, s4.z, s4.w, b == 0 ? ylo5 : ec[0].a};
            const T nw[5] = {n4.x, n4.y, n4.z, n4.w, b == 0 ? ec[1].a : yhi5};
            const T mv[5] = {xm[b].x, xm[b].y, xm[b].z, xm[b].w, em[b].a};
            const T uv[5] = {xp[b].x, xp[b].y, xp[b].z, xp[b].w, ep[b].a};
            const T rv[5] = {rh[b].x, rh[b].y, rh[b].z, rh[b].w, h5[b]};
            T left = __shfl_up(cv[3], 1, LANES), right = __shfl_down(cv[0], 1, LANES);
            if (lane == 0) left = ec[b].a;                    // 0 at the wall (no edge pair)
            if (lane == LANES - 1) right = ec[b].a;
            // x neighbours of the five nodes: node u's -x one is wxn[u], its +x one exn[u]
            const T wxn[5] = {left, cv[0], cv[1], cv[2], cv[3]};
            const T exn[5] = {cv[1], cv[2], cv[3], right, ec[b].b};
            T r[5];
#pragma unroll
            for (int u = 0; u < (FIFTH ? 5 : 4); ++u)
                r[u] = mg_reg_resid(rv[u], cv[u], wxn[u], exn[u], sv[u], nw[u], mv[u], uv[u], kax[u], kbx[u],
                                    kcx[u], kay[b], kby[b], kcy[b], za, zb, zc);
            // solid or irregular nodes: their residual from ri (0 at a solid node)
            const T qv[5] = {ri4[b].x, ri4[b].y, ri4[b].z, ri4[b].w, ri5[b]};
#pragma unroll
            for (int u = 0; u < (FIFTH ? 5 : 4); ++u) r[u] = ((sk[b] >> u) & 1u) ? qv[u] : r[u];
            const bool live = pv && rok[b];
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = (live && u < nv) ? r[u] : T(0);
            T v4 = __shfl_down(r[0], 1, LANES);
            if (lane == LANES - 1) v4 = (FIFTH && live && need5) ? r[4] : T(0);
            xr[b][0] = w0[0] * r[0] + w0[1] * r[1] + w0[2] * r[2];
            xr[b][1] = w1[0] * r[2] + w1[1] * r[3] + w1[2] * v4;
        }
        if (p & 1) {
            // fine plane 2K + 1: the last of coarse plane K, the first of K + 1
            const int K = (p - 1) >> 1;
            if (K >= K0) {
                add_plane(K, 2, xr);
                emit(K);
            }
            if (K + 1 < K1) {
                open(K + 1);
                add_plane(K + 1, 0, xr);
            }
        } else {
            add_plane(p >> 1, 1, xr);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            xm[b] = xc[b];
            xc[b] = xp[b];
            em[b] = ec[b];
            ec[b] = ep[b];
        }
    }
}

// 1 / d of a diagonal that reciprocals_normal has let through: the hardware's reciprocal and a Newton
// step in FP32, a third of the instructions of a division.  c2 r (1 / d) rounds once more than
// c2 r / d: FP32 V-cycles of six grids of 10 to 27 M nodes differ from FP64 by 1.9e-7 .. 2.9e-7 in the
// 2-norm with either.
__device__ __forceinline__ float recip(float d)
{
    const float r = __builtin_amdgcn_rcpf(d);
    return __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
}
__device__ __forceinline__ double recip(double d) { return 1.0 / d; }

// Two smoothing steps from x_0 in one pass over memory (a post-smoothing pass of nu = 2):
//   y = x_0 + c2a (rho - K x_0) / diag K,  z = y + c1 (y - x_0) + c2 (rho - K y) / diag K
// with y never stored: x_0 and rho in, z out, 3 vectors instead of 7.  A block marches in z over
// 2 Pair::waves rows of a 256-node segment: wavefront w forms y of its two rows at plane k (four
// nodes per lane, x of the planes k - 1 .. k + 1 in registers), then z at plane k - 1 from the y
// of planes k - 2 .. k; the rows of the neighbouring wavefronts come through LDS, one barrier a
// plane.  The block's first and last row and a chunk's outer planes are formed for y alone.
// Where a row has more segments (SEG), the outer lanes form y at the node beyond theirs as well.
// Irregular nodes: y is read from yi (0 at the solid nodes), z is not written; k_mg_pair_irregular
// forms both, before.
// A block's waves fill a CU's registers: 12 in FP32, 8 in FP64; 1 / diag K is formed once for both
// steps.  Bound by its few wavefronts (registers; 2.6 a SIMD in FP32, which wait half of their time)
// and the vector instructions of the two steps (half of the cycles).  Measured with k_mg_pair_irregular, against the two sweeps (us): 256^3 FP32 48 + 8 against
// 41 + 48, FP64 109 + 9 against 90 + 119; 512^3 FP32 473 + 25 against 393 + 491.
template <typename T>
struct Pair {
    static constexpr int waves = sizeof(T) == 4 ? 12 : 8, rows = 2 * waves - 2;   // rows stored by a block
};
template <typename T, bool SEG>
__global__ void __launch_bounds__(64 * Pair<T>::waves)
    k_mg_pair(Geom g, Tiling tl, Coef<T> cf, const uint32_t *__restrict__ skip, const T *__restrict__ x,
              const T *__restrict__ rho, const T *__restrict__ yi, T *__restrict__ out, T c2a, T c1, T c2,
              const DevState *st)
{
    using V = typename MgVec4<T>::type;
    constexpr int PAIR_WAVES = Pair<T>::waves, PAIR_ROWS = Pair<T>::rows;
    __shared__ V sh[2][PAIR_WAVES][2][64];                    // y of a plane's rows
    if (st && st->done) return;
    int bs, by, bz;
    if (!tile_of_block(tl, (int)blockIdx.x, bs, by, bz)) return;
    const int wv = (int)threadIdx.y, lane = (int)threadIdx.x;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const size_t plane = (size_t)nx * ny, wplane = (size_t)ny * g.W;
    const int i0 = 1 + 256 * bs + 4 * lane;
    const int nv = min(4, nx - 1 - i0);                       // interior nodes of the lane
    const int ic = min(i0, nx - 1);                           // lanes past the row end: the wall node
    const bool needr = SEG && lane == 63 && i0 + 4 <= nx - 2; // the node beyond the lane's is interior
    const bool needl = SEG && lane == 0 && bs > 0;
    const bool edge = needr || needl;
    const int ie = needr ? i0 + 4 : (needl ? i0 - 1 : ic);    // that node
    const uint32_t past = 0xFu & ~((1u << max(nv, 0)) - 1u);  // the lane's places past the row end
    const uint32_t eoff = (uint32_t)((needr ? 4 : -2) * (int)sizeof(T)), hoff = (uint32_t)((ie - ic) * (int)sizeof(T));
    T kax[5], kbx[5], kcx[5];
    {
        const T *x5 = cf.xs + (size_t)5 * cf.xp, *x6 = x5 + cf.xp, *x7 = x6 + cf.xp;
        const V va = *reinterpret_cast<const V *>(x5 + ic), vb = *reinterpret_cast<const V *>(x6 + ic),
                vc = *reinterpret_cast<const V *>(x7 + ic);
        const T a[5] = {va.x, va.y, va.z, va.w, SEG ? x5[ie] : T(0)}, bb[5] = {vb.x, vb.y, vb.z, vb.w, SEG ? x6[ie] : T(1)},
                c[5] = {vc.x, vc.y, vc.z, vc.w, SEG ? x7[ie] : T(0)};
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            kax[u] = a[u];
            kbx[u] = bb[u];
            kcx[u] = c[u];
        }
    }
    // the wavefront's rows j0, j0 + 1, and byte offsets of node ic on x rows j0 - 1 .. j0 + 2
    // (clamped to the wall rows, where x is 0); rows outside the interior have y = 0
    const int j0 = PAIR_ROWS * by + 2 * wv;
    uint32_t ox[4], ow[2];
#pragma unroll
    for (int c = 0; c < 4; ++c) ox[c] = (uint32_t)((ic + nx * min(max(j0 - 1 + c, 0), ny - 1)) * sizeof(T));
    bool rok[2], own[2];
    T kay[2], kby[2], kcy[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int j = j0 + b, jc = min(j, ny - 1);
        rok[b] = j >= 1 && j <= ny - 2;
        own[b] = rok[b] && 2 * wv + b >= 1 && 2 * wv + b <= PAIR_ROWS;
        ow[b] = (uint32_t)((jc * g.W + (ic >> 5)) * sizeof(uint32_t));
        kay[b] = wave_uniform(cf.c[1][8 * jc + 5]);
        kby[b] = wave_uniform(cf.c[1][8 * jc + 6]);
        kcy[b] = wave_uniform(cf.c[1][8 * jc + 7]);
    }
    const int K0 = 1 + bz * tl.TZ, K1 = min(K0 + tl.TZ, nz - 1);
    // x at the plane behind (m) and the current one (c) with the edge pairs; y of the two planes
    // behind (0, 1), at the edge node too; rho, 1 / diag K and the skip bits of the plane behind
    V xm[2], xc[2], y0[2], y1[2], rp[2], dp[2];
    MgPair<T> em[2], ec[2];
    T ye1[2] = {T(0), T(0)};
    uint32_t skp[2] = {0u, 0u}, skn[2];
    const V zero4 = V{T(0), T(0), T(0), T(0)};
    auto skip_bits = [&](int q, int b) -> uint32_t {
        const uint64_t pair = bload_u64(plane_rsrc(skip + (size_t)q * wplane), ow[b]);
        const uint32_t m = (uint32_t)(pair >> (ic & 31)) & ((1u << max(nv, 0)) - 1u);
        if (!SEG || !edge) return m;
        return m | (needr ? ((uint32_t)(pair >> (ic & 31)) & 0x10u) : (((uint32_t)(pair >> ((ic & 31) - 1)) & 1u) << 4));
    };
    {
        const __amdgpu_buffer_rsrc_t xb = plane_rsrc(x + (size_t)max(K0 - 2, 0) * plane),
                                     xk = plane_rsrc(x + (size_t)(K0 - 1) * plane);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            skn[b] = skip_bits(K0 - 1, b);
            xm[b] = bload4<T>(xb, ox[b + 1]);
            xc[b] = bload4<T>(xk, ox[b + 1]);
            em[b] = edge ? bload2<T>(xb, ox[b + 1] + eoff) : MgPair<T>{T(0), T(0)};
            ec[b] = edge ? bload2<T>(xk, ox[b + 1] + eoff) : MgPair<T>{T(0), T(0)};
            y0[b] = y1[b] = rp[b] = dp[b] = zero4;
        }
    }
    for (int k = K0 - 1; k <= K1; ++k) {
        const size_t kp = (size_t)k * plane;
        const __amdgpu_buffer_rsrc_t xk = plane_rsrc(x + kp), xn = plane_rsrc(x + (size_t)min(k + 1, nz - 1) * plane);
        const __amdgpu_buffer_rsrc_t rk = plane_rsrc(rho + kp), yk = plane_rsrc(yi + kp);
        V xp[2], rh[2], yi4[2];
        MgPair<T> ep[2];
        uint32_t sk[2];
        T h5[2], yi5[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const uint32_t o = ox[b + 1];
            sk[b] = skn[b];
            skn[b] = skip_bits(min(k + 1, nz - 1), b);
            xp[b] = bload4<T>(xn, o);
            rh[b] = bload4<T>(rk, o);
            // y at the lane's solid and irregular nodes (issued with the other loads)
            if (sk[b]) yi4[b] = bload4<T>(yk, o);
            else yi4[b] = zero4;
            yi5[b] = (SEG && (sk[b] & 0x10u)) ? bload1<T>(yk, o + hoff) : T(0);
            ep[b] = edge ? bload2<T>(xn, o + eoff) : MgPair<T>{T(0), T(0)};
            h5[b] = edge ? bload1<T>(rk, o + hoff) : T(0);
        }
        // the outer y neighbours: x rows j0 - 1 and j0 + 2
        const V xlo = bload4<T>(xk, ox[0]), xhi = bload4<T>(xk, ox[3]);
        const T xlo5 = edge ? bload1<T>(xk, ox[0] + hoff) : T(0), xhi5 = edge ? bload1<T>(xk, ox[3] + hoff) : T(0);
        V y2[2], dk[2];
        T ye2[2];
        {
            const T *cz = cf.c[2] + 8 * k;
            const T za = wave_uniform(cz[5]), zb = wave_uniform(cz[6]), zc = wave_uniform(cz[7]);
            const bool pv = k >= 1 && k <= nz - 2;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const T ce = needr ? ec[b].a : ec[b].b, co = needr ? ec[b].b : ec[b].a;   // edge node, the one beyond
                const T me = needr ? em[b].a : em[b].b, pe = needr ? ep[b].a : ep[b].b;
                const V &s4 = b == 0 ? xlo : xc[0];
                const V &n4 = b == 0 ? xc[1] : xhi;
                const T se = b == 0 ? xlo5 : (needr ? ec[0].a : ec[0].b);
                const T ne = b == 0 ? (needr ? ec[1].a : ec[1].b) : xhi5;
                const T cv[4] = {xc[b].x, xc[b].y, xc[b].z, xc[b].w};
                const T sv[4] = {s4.x, s4.y, s4.z, s4.w}, nw[4] = {n4.x, n4.y, n4.z, n4.w};
                const T mv[4] = {xm[b].x, xm[b].y, xm[b].z, xm[b].w}, uv[4] = {xp[b].x, xp[b].y, xp[b].z, xp[b].w};
                const T rv[4] = {rh[b].x, rh[b].y, rh[b].z, rh[b].w}, iv[4] = {yi4[b].x, yi4[b].y, yi4[b].z, yi4[b].w};
                T left = __shfl_up(cv[3], 1, 64), right = __shfl_down(cv[0], 1, 64);
                if (lane == 0) left = needl ? ce : T(0);
                if (lane == 63) right = needr ? ce : T(0);
                const bool live = pv && rok[b];               // uniform
                T yv[4], dv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const T r = mg_reg_resid(rv[u], cv[u], u == 0 ? left : cv[u - 1], u == 3 ? right : cv[u + 1], sv[u],
                                             nw[u], mv[u], uv[u], kax[u], kbx[u], kcx[u], kay[b], kby[b], kcy[b], za, zb, zc);
                    dv[u] = recip(kbx[u] + kby[b] + zb);
                    yv[u] = cv[u] + c2a * r * dv[u];
                }
                if (__any(sk[b] | past)) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if ((sk[b] >> u) & 1u) yv[u] = iv[u];
                        if ((past >> u) & 1u) yv[u] = T(0);
                    }
                }
                y2[b] = live ? V{yv[0], yv[1], yv[2], yv[3]} : zero4;
                dk[b] = V{dv[0], dv[1], dv[2], dv[3]};
                ye2[b] = T(0);
                if (SEG) {
                    const T r = mg_reg_resid(h5[b], ce, needr ? cv[3] : co, needr ? co : cv[0], se, ne, me, pe, kax[4], kbx[4],
                                             kcx[4], kay[b], kby[b], kcy[b], za, zb, zc);
                    ye2[b] = ce + c2a * r / (kbx[4] + kby[b] + zb);
                    if (sk[b] & 0x10u) ye2[b] = yi5[b];
                    if (!live || !edge) ye2[b] = T(0);
                }
            }
        }
        if (k >= K0 + 1) {
            const int q = k - 1;
            const T *cz = cf.c[2] + 8 * q;
            const T za = wave_uniform(cz[5]), zb = wave_uniform(cz[6]), zc = wave_uniform(cz[7]);
            const V ylo = wv > 0 ? sh[q & 1][wv - 1][1][lane] : zero4;
            const V yhi = wv < PAIR_WAVES - 1 ? sh[q & 1][wv + 1][0][lane] : zero4;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const V &s4 = b == 0 ? ylo : y1[0];
                const V &n4 = b == 0 ? y1[1] : yhi;
                const T cv[4] = {y1[b].x, y1[b].y, y1[b].z, y1[b].w};
                const T sv[4] = {s4.x, s4.y, s4.z, s4.w}, nw[4] = {n4.x, n4.y, n4.z, n4.w};
                const T mv[4] = {y0[b].x, y0[b].y, y0[b].z, y0[b].w}, uv[4] = {y2[b].x, y2[b].y, y2[b].z, y2[b].w};
                const T dv[4] = {dp[b].x, dp[b].y, dp[b].z, dp[b].w};
                const T rv[4] = {rp[b].x, rp[b].y, rp[b].z, rp[b].w}, xv[4] = {xm[b].x, xm[b].y, xm[b].z, xm[b].w};
                T left = __shfl_up(cv[3], 1, 64), right = __shfl_down(cv[0], 1, 64);
                if (lane == 0) left = ye1[b];                  // 0 at a wall
                if (lane == 63) right = ye1[b];
                T zv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const T r = mg_reg_resid(rv[u], cv[u], u == 0 ? left : cv[u - 1], u == 3 ? right : cv[u + 1], sv[u],
                                             nw[u], mv[u], uv[u], kax[u], kbx[u], kcx[u], kay[b], kby[b], kcy[b], za, zb, zc);
                    zv[u] = cv[u] + c1 * (cv[u] - xv[u]) + c2 * r * dv[u];
                }
                if (own[b]) {
                    T *o = out + (size_t)q * plane + (ox[b + 1] / (uint32_t)sizeof(T));
                    if (nv == 4 && (skp[b] & 0xFu) == 0u) {
                        *reinterpret_cast<V *>(o) = V{zv[0], zv[1], zv[2], zv[3]};
                    } else {
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (u < nv && !((skp[b] >> u) & 1u)) o[u] = zv[u];
                    }
                }
            }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            sh[k & 1][wv][b][lane] = y2[b];
            xm[b] = xc[b];
            xc[b] = xp[b];
            em[b] = ec[b];
            ec[b] = ep[b];
            y0[b] = y1[b];
            y1[b] = y2[b];
            ye1[b] = ye2[b];
            rp[b] = rh[b];
            dp[b] = dk[b];
            skp[b] = sk[b];
        }
        __syncthreads();
    }
}

// The second smoothing step from zero, x_2 = x_1 + c1 x_1 + c2 (rho - K x_1) / diag K, with
// x_1 = c2a rho / diag K formed here instead of stored and read: rho in, x_2 out, 2 vectors instead
// of 3, and the vector update before it writes one less.  The march of k_mg_pair, with x_1 of a
// plane's rows in place of y.  x_1 holds the step at the irregular nodes and 0 at the solid ones;
// the irregular rows run in the blocks after the tiles, eight lanes a row.  Bound as k_mg_pair is (3.5
// wavefronts a SIMD, waiting 62 % of their time; vector ALUs busy in 54 % of the cycles).
// Measured against the stored x_1 (us, this step / the two vector updates before it): 256^3 FP32
// 41 / 50 + 34 against 45 / 63 + 48, FP64 88 / 113 + 80 against 100 / 145 + 109; 512^3 FP32
// 352 / 440 + 321 against 393 / 576 + 452.  Loading a plane ahead costs 5 to 15 %, as in the other
// marches: registers.
template <typename T>
struct Second {
    static constexpr int waves = 8, rows = 2 * waves - 2;     // rows stored by a block
};
template <typename T, bool SEG>
__global__ void __launch_bounds__(64 * Second<T>::waves)
    k_mg_second(Geom g, Tiling tl, Coef<T> cf, Irr<T> ir, const uint32_t *__restrict__ skip, const T *__restrict__ x1,
                const T *__restrict__ rho, T *__restrict__ out, T c2a, T c1, T c2, const DevState *st)
{
    using V = typename MgVec4<T>::type;
    constexpr int WAVES = Second<T>::waves, ROWS = Second<T>::rows;
    __shared__ V sh[2][WAVES][2][64];                         // x_1 of a plane's rows
    if (st && st->done) return;
    const int wv = (int)threadIdx.y, lane = (int)threadIdx.x;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const size_t plane = (size_t)nx * ny, wplane = (size_t)ny * g.W;
    if ((int)blockIdx.x >= tl.nblk) {
        const int t = ((int)blockIdx.x - tl.nblk) * 64 * WAVES + 64 * wv + lane, q = t & 7, row = t >> 3;
        const int rc = min(row, ir.n - 1), e = ir.node[rc];
        const T kq = ir.k7[7 * (size_t)rc + min(q, 6)], kd0 = ir.k7[7 * (size_t)rc], rho0 = rho[e];
        const int k0 = e / (int)plane, r0 = e - k0 * (int)plane, j0 = r0 / nx, i0 = r0 - j0 * nx;
        const int i = i0 + (q == 2) - (q == 1), j = j0 + (q == 4) - (q == 3), k = k0 + (q == 6) - (q == 5);
        const bool wall = i == 0 || i == nx - 1 || j == 0 || j == ny - 1 || k == 0 || k == nz - 1;
        const size_t eq = (size_t)i + (size_t)nx * j + plane * k;
        const bool sb = (skip[((size_t)j + (size_t)ny * k) * g.W + (i >> 5)] >> (i & 31)) & 1u;
        const T a = x1[eq], b = rho[eq], d = cf.c[0][8 * i + 6] + cf.c[1][8 * j + 6] + cf.c[2][8 * k + 6];
        const T y = wall ? T(0) : (sb ? a : c2a * b / d);
        T sum = q < 7 ? kq * y : T(0);
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) sum += __shfl_xor(sum, o, 64);
        if (q == 0 && row < ir.n) out[e] = y + c1 * y + c2 * (rho0 - sum) / kd0;
        return;
    }
    int bs, by, bz;
    if (!tile_of_block(tl, (int)blockIdx.x, bs, by, bz)) return;
    const int i0 = 1 + 256 * bs + 4 * lane;
    const int nv = min(4, nx - 1 - i0);                       // interior nodes of the lane
    const int ic = min(i0, nx - 1);                           // lanes past the row end: the wall node
    const bool needr = SEG && lane == 63 && i0 + 4 <= nx - 2; // the node beyond the lane's is interior
    const bool needl = SEG && lane == 0 && bs > 0;
    const bool edge = needr || needl;
    const int ie = needr ? i0 + 4 : (needl ? i0 - 1 : ic);    // that node
    const uint32_t past = 0xFu & ~((1u << max(nv, 0)) - 1u);  // the lane's places past the row end
    const uint32_t hoff = (uint32_t)((ie - ic) * (int)sizeof(T));
    T kax[4], kbx[5], kcx[4];
    {
        const T *x5 = cf.xs + (size_t)5 * cf.xp, *x6 = x5 + cf.xp, *x7 = x6 + cf.xp;
        const V va = *reinterpret_cast<const V *>(x5 + ic), vb = *reinterpret_cast<const V *>(x6 + ic),
                vc = *reinterpret_cast<const V *>(x7 + ic);
        const T a[4] = {va.x, va.y, va.z, va.w}, bb[5] = {vb.x, vb.y, vb.z, vb.w, SEG ? x6[ie] : T(1)},
                c[4] = {vc.x, vc.y, vc.z, vc.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            kax[u] = a[u];
            kcx[u] = c[u];
        }
#pragma unroll
        for (int u = 0; u < 5; ++u) kbx[u] = bb[u];
    }
    // the wavefront's rows j0, j0 + 1 (rows outside the interior have x_1 = 0)
    const int j0 = ROWS * by + 2 * wv;
    uint32_t ox[2], ow[2];
    bool rok[2], own[2];
    T kay[2], kby[2], kcy[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int j = j0 + b, jc = min(j, ny - 1);
        rok[b] = j >= 1 && j <= ny - 2;
        own[b] = rok[b] && 2 * wv + b >= 1 && 2 * wv + b <= ROWS;
        ox[b] = (uint32_t)((ic + nx * jc) * sizeof(T));
        ow[b] = (uint32_t)((jc * g.W + (ic >> 5)) * sizeof(uint32_t));
        kay[b] = wave_uniform(cf.c[1][8 * jc + 5]);
        kby[b] = wave_uniform(cf.c[1][8 * jc + 6]);
        kcy[b] = wave_uniform(cf.c[1][8 * jc + 7]);
    }
    const int K0 = 1 + bz * tl.TZ, K1 = min(K0 + tl.TZ, nz - 1);
    // x_1 of the two planes behind (0, 1), at the edge node too; rho, 1 / diag K and the skip bits
    // of the plane behind
    V y0[2], y1[2], rp[2], dp[2];
    T ye1[2] = {T(0), T(0)};
    uint32_t skp[2] = {0u, 0u}, skn[2];
    const V zero4 = V{T(0), T(0), T(0), T(0)};
    auto skip_bits = [&](int q, int b) -> uint32_t {
        const uint64_t pair = bload_u64(plane_rsrc(skip + (size_t)q * wplane), ow[b]);
        const uint32_t m = (uint32_t)(pair >> (ic & 31)) & ((1u << max(nv, 0)) - 1u);
        if (!SEG || !edge) return m;
        return m | (needr ? ((uint32_t)(pair >> (ic & 31)) & 0x10u) : (((uint32_t)(pair >> ((ic & 31) - 1)) & 1u) << 4));
    };
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        y0[b] = y1[b] = rp[b] = dp[b] = zero4;
        skn[b] = skip_bits(K0 - 1, b);
    }
    for (int k = K0 - 1; k <= K1; ++k) {
        const __amdgpu_buffer_rsrc_t rk = plane_rsrc(rho + (size_t)k * plane), yk = plane_rsrc(x1 + (size_t)k * plane);
        V rh[2], yi4[2];
        uint32_t sk[2];
        T h5[2], yi5[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            sk[b] = skn[b];
            skn[b] = skip_bits(min(k + 1, nz - 1), b);
            rh[b] = bload4<T>(rk, ox[b]);
            h5[b] = edge ? bload1<T>(rk, ox[b] + hoff) : T(0);
            // x_1 at the lane's solid and irregular nodes
            if (sk[b]) yi4[b] = bload4<T>(yk, ox[b]);
            else yi4[b] = zero4;
            yi5[b] = (SEG && (sk[b] & 0x10u)) ? bload1<T>(yk, ox[b] + hoff) : T(0);
        }
        V y2[2], dk[2];
        T ye2[2];
        {
            const T zb = wave_uniform(cf.c[2][8 * k + 6]);
            const bool pv = k >= 1 && k <= nz - 2;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const T rv[4] = {rh[b].x, rh[b].y, rh[b].z, rh[b].w}, iv[4] = {yi4[b].x, yi4[b].y, yi4[b].z, yi4[b].w};
                const bool live = pv && rok[b];               // uniform
                T yv[4], dv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    dv[u] = recip(kbx[u] + kby[b] + zb);
                    yv[u] = c2a * rv[u] * dv[u];
                }
                if (__any(sk[b] | past)) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if ((sk[b] >> u) & 1u) yv[u] = iv[u];
                        if ((past >> u) & 1u) yv[u] = T(0);
                    }
                }
                y2[b] = live ? V{yv[0], yv[1], yv[2], yv[3]} : zero4;
                dk[b] = V{dv[0], dv[1], dv[2], dv[3]};
                ye2[b] = T(0);
                if (SEG && live && edge) ye2[b] = (sk[b] & 0x10u) ? yi5[b] : c2a * h5[b] / (kbx[4] + kby[b] + zb);
            }
        }
        if (k >= K0 + 1) {
            const int q = k - 1;
            const T *cz = cf.c[2] + 8 * q;
            const T za = wave_uniform(cz[5]), zb = wave_uniform(cz[6]), zc = wave_uniform(cz[7]);
            const V ylo = wv > 0 ? sh[q & 1][wv - 1][1][lane] : zero4;
            const V yhi = wv < WAVES - 1 ? sh[q & 1][wv + 1][0][lane] : zero4;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const V &s4 = b == 0 ? ylo : y1[0];
                const V &n4 = b == 0 ? y1[1] : yhi;
                const T cv[4] = {y1[b].x, y1[b].y, y1[b].z, y1[b].w}, dv[4] = {dp[b].x, dp[b].y, dp[b].z, dp[b].w};
                const T sv[4] = {s4.x, s4.y, s4.z, s4.w}, nw[4] = {n4.x, n4.y, n4.z, n4.w};
                const T mv[4] = {y0[b].x, y0[b].y, y0[b].z, y0[b].w}, uv[4] = {y2[b].x, y2[b].y, y2[b].z, y2[b].w};
                const T rv[4] = {rp[b].x, rp[b].y, rp[b].z, rp[b].w};
                T left = __shfl_up(cv[3], 1, 64), right = __shfl_down(cv[0], 1, 64);
                if (lane == 0) left = ye1[b];                  // 0 at a wall
                if (lane == 63) right = ye1[b];
                T zv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const T r = mg_reg_resid(rv[u], cv[u], u == 0 ? left : cv[u - 1], u == 3 ? right : cv[u + 1], sv[u],
                                             nw[u], mv[u], uv[u], kax[u], kbx[u], kcx[u], kay[b], kby[b], kcy[b], za, zb, zc);
                    zv[u] = cv[u] + c1 * cv[u] + c2 * r * dv[u];
                }
                if (own[b]) {
                    T *o = out + (size_t)q * plane + (ox[b] / (uint32_t)sizeof(T));
                    if (nv == 4 && (skp[b] & 0xFu) == 0u) {
                        *reinterpret_cast<V *>(o) = V{zv[0], zv[1], zv[2], zv[3]};
                    } else {
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (u < nv && !((skp[b] >> u) & 1u)) o[u] = zv[u];
                    }
                }
            }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            sh[k & 1][wv][b][lane] = y2[b];
            y0[b] = y1[b];
            y1[b] = y2[b];
            ye1[b] = ye2[b];
            rp[b] = rh[b];
            dp[b] = dk[b];
            skp[b] = sk[b];
        }
        __syncthreads();
    }
}

// The irregular rows of k_mg_pair: y and z at the irregular nodes, yi and out.  Eight lanes take
// a row: lane q forms y at the row's q-th node (its own, then the -x, +x, -y, +y, -z, +z
// neighbours) from x_0.  Bound by its gathers.
template <typename T>
__global__ void __launch_bounds__(NT) k_mg_pair_irregular(Geom g, Coef<T> cf, Irr<T> ir,
                                                          const uint32_t *__restrict__ skip, const T *__restrict__ x,
                                                          const T *__restrict__ rho, T *__restrict__ yi,
                                                          T *__restrict__ out, T c2a, T c1, T c2, const DevState *st)
{
    const int done = st ? st->done : 0;
    const int t = (int)(blockIdx.x * NT + threadIdx.x), q = t & 7;
    const bool live = (t >> 3) < ir.n;
    const int row = min(t >> 3, ir.n - 1);
    const int nx = g.nx, ny = g.ny, nz = g.nz, plane = nx * ny;
    const int e = ir.node[row];
    const T kq = ir.k7[7 * (size_t)row + min(q, 6)], kd0 = ir.k7[7 * (size_t)row], x0 = x[e], rho0 = rho[e];
    const int k0 = e / plane, r0 = e - k0 * plane, j0 = r0 / nx, i0 = r0 - j0 * nx;
    const int i = i0 + (q == 2) - (q == 1), j = j0 + (q == 4) - (q == 3), k = k0 + (q == 6) - (q == 5);
    T y = T(0);
    const bool wall = i == 0 || i == nx - 1 || j == 0 || j == ny - 1 || k == 0 || k == nz - 1;
    if (!wall && q < 7) {
        const size_t w = ((size_t)j + (size_t)ny * k) * g.W + (i >> 5);
        const bool sb = (skip[w] >> (i & 31)) & 1u, ib = (ir.bits[w] >> (i & 31)) & 1u;
        const size_t eq = (size_t)i + (size_t)nx * j + (size_t)plane * k;
        const T c = x[eq], xw = x[eq - 1], xe = x[eq + 1], xs = x[eq - nx], xn = x[eq + nx], xd = x[eq - plane],
                xu = x[eq + plane], rq = rho[eq];
        T a[7] = {cf.c[0][8 * i + 6] + cf.c[1][8 * j + 6] + cf.c[2][8 * k + 6], cf.c[0][8 * i + 5], cf.c[0][8 * i + 7],
                  cf.c[1][8 * j + 5], cf.c[1][8 * j + 7], cf.c[2][8 * k + 5], cf.c[2][8 * k + 7]};
        if (ib) {
            const T *k7 = ir.k7 + 7 * (size_t)irr_row_of(ir, w, i);
#pragma unroll
            for (int v = 0; v < 7; ++v) a[v] = k7[v];
        }
        const T kx = a[0] * c + a[1] * xw + a[2] * xe + a[3] * xs + a[4] * xn + a[5] * xd + a[6] * xu;
        if (!sb || ib) y = c + c2a * (rq - kx) / a[0];
    }
    T sum = q < 7 ? kq * y : T(0);
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) sum += __shfl_xor(sum, o, 64);
    if (q != 0 || !live || done) return;
    yi[e] = y;
    out[e] = y + c1 * (y - x0) + c2 * (rho0 - sum) / kd0;
}

// The same on small grids, whose march is bound by the round trips of its planes: a wavefront forms
// the residual of one fine plane p = 2K - 1 + q for coarse plane K, all its loads issued at once,
// and the three wavefronts of a coarse plane sum their shares through LDS.  Lanes take the groups
// of four fine nodes of a plane's coarse rows in order, whatever the row length; of a wavefront's
// 64 groups the inner 62 are summed, so that both x neighbours and the fifth fine point always
// come from the adjacent lanes.  Fine rows and planes shared by two coarse ones are formed twice.
constexpr int RRS_WAVE = 62, RRS_WAVES = 2;                    // groups of a wavefront, wavefronts per plane
template <typename T>
__global__ void __launch_bounds__(64 * 3 * RRS_WAVES)
    k_mg_resid_restrict_short(Geom g, Coef<T> cf, const uint32_t *__restrict__ skip, const T *__restrict__ x,
                              const T *__restrict__ rho, const T *__restrict__ ri, int ncx, int ncy, int ncz,
                              MgAxis<T> ax, MgAxis<T> ay, MgAxis<T> az, int gpr, int nbx, T *__restrict__ rc,
                              MgFirst<T> F, const DevState *st)
{
    using V = typename MgVec4<T>::type;
    __shared__ T sh[RRS_WAVES][2][2][64];                      // the shares of planes q = 1, 2
    const int done = st ? st->done : 0;                        // used before the stores: nothing waits for it
    const int per = (int)gridDim.x / NXCD, blk = ((int)blockIdx.x % NXCD) * per + (int)blockIdx.x / NXCD;
    const int K = 1 + blk / nbx;
    if (K > ncz - 2) return;                                   // whole block
    const int lane = (int)threadIdx.x, q = (int)threadIdx.y, w = (int)threadIdx.z;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int item = ((blk % nbx) * RRS_WAVES + w) * RRS_WAVE + lane - 1;
    const int items = gpr * (ncy - 2), it = min(max(item, 0), items - 1);
    const int J = 1 + it / gpr, gx = it % gpr, I0 = 1 + 2 * gx, f0 = 4 * gx + 1;
    const bool live = lane >= 1 && lane <= RRS_WAVE && item < items;
    const bool own0 = live && I0 <= ncx - 2, own1 = live && I0 + 1 <= ncx - 2;
    const int nv = min(4, nx - 1 - f0);                        // interior fine nodes of the group
    const int p = 2 * K - 1 + q, pc = min(p, nz - 1);
    const size_t plane = (size_t)nx * ny;
    int row[5];                                                // fine rows 2J - 2 .. 2J + 2 (the wall row beyond)
#pragma unroll
    for (int c = 0; c < 5; ++c) row[c] = f0 + nx * min(2 * J - 2 + c, ny - 1);
    uint64_t pair[3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
        __builtin_memcpy(&pair[b], skip + ((size_t)min(2 * J - 1 + b, ny - 1) + (size_t)ny * pc) * g.W + (f0 >> 5), 8);
    const T *xk = x + plane * pc, *xm = x + plane * (p - 1), *xu = x + plane * min(p + 1, nz - 1);
    V c4[5], m4[3], u4[3], r4[3], i4[3];
#pragma unroll
    for (int c = 0; c < 5; ++c) c4[c] = *reinterpret_cast<const V *>(xk + row[c]);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        m4[b] = *reinterpret_cast<const V *>(xm + row[b + 1]);
        u4[b] = *reinterpret_cast<const V *>(xu + row[b + 1]);
        r4[b] = *reinterpret_cast<const V *>(rho + plane * pc + row[b + 1]);
    }
    T ka[4], kb[4], kc[4], ky[3][3], wx0[3], wx1[3], wy[3];
    {
        const T *x5 = cf.xs + (size_t)5 * cf.xp + f0, *x6 = x5 + cf.xp, *x7 = x6 + cf.xp;
        const V va = *reinterpret_cast<const V *>(x5), vb = *reinterpret_cast<const V *>(x6),
                vc = *reinterpret_cast<const V *>(x7);
        const T a[4] = {va.x, va.y, va.z, va.w}, bb[4] = {vb.x, vb.y, vb.z, vb.w}, c[4] = {vc.x, vc.y, vc.z, vc.w};
        const int a0 = own0 ? I0 : 1, a1 = own1 ? I0 + 1 : a0;
#pragma unroll
        for (int u = 0; u < 4; ++u) { ka[u] = a[u]; kb[u] = bb[u]; kc[u] = c[u]; }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
#pragma unroll
            for (int d = 0; d < 3; ++d) ky[b][d] = cf.c[1][8 * min(2 * J - 1 + b, ny - 1) + 5 + d];
            wx0[b] = ax.rw[3 * a0 + b];
            wx1[b] = ax.rw[3 * a1 + b];
            wy[b] = ay.rw[3 * J + b];
        }
    }
    const T za = cf.c[2][8 * pc + 5], zb = cf.c[2][8 * pc + 6], zc = cf.c[2][8 * pc + 7], wz = az.rw[3 * K + q];
    T dg[2] = {T(0), T(0)};
    const size_t e = (size_t)I0 + (size_t)ncx * (J + (size_t)ncy * K);
    if (q == 0) {
        if (own0) dg[0] = F.diag[e];
        if (own1) dg[1] = F.diag[e + 1];
    }
    uint32_t sk[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        sk[b] = (uint32_t)(pair[b] >> (f0 & 31)) & ((1u << nv) - 1u);
        i4[b] = V{T(0), T(0), T(0), T(0)};
        if (sk[b]) i4[b] = *reinterpret_cast<const V *>(ri + plane * pc + row[b + 1]);
    }
    T s0 = T(0), s1 = T(0);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const bool ok = p <= nz - 2 && 2 * J - 1 + b <= ny - 2;
        const T cv[4] = {c4[b + 1].x, c4[b + 1].y, c4[b + 1].z, c4[b + 1].w};
        const T sv[4] = {c4[b].x, c4[b].y, c4[b].z, c4[b].w}, nw[4] = {c4[b + 2].x, c4[b + 2].y, c4[b + 2].z, c4[b + 2].w};
        const T mv[4] = {m4[b].x, m4[b].y, m4[b].z, m4[b].w}, uv[4] = {u4[b].x, u4[b].y, u4[b].z, u4[b].w};
        const T rv[4] = {r4[b].x, r4[b].y, r4[b].z, r4[b].w}, iv[4] = {i4[b].x, i4[b].y, i4[b].z, i4[b].w};
        T left = __shfl_up(cv[3], 1, 64), right = __shfl_down(cv[0], 1, 64);
        if (gx == 0) left = T(0);                              // the walls
        if (gx == gpr - 1) right = T(0);
        T r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T wv = u == 0 ? left : cv[u - 1], ev = u == 3 ? right : cv[u + 1];
            r[u] = mg_reg_resid(rv[u], cv[u], wv, ev, sv[u], nw[u], mv[u], uv[u], ka[u], kb[u], kc[u], ky[b][0],
                                ky[b][1], ky[b][2], za, zb, zc);
            if ((sk[b] >> u) & 1u) r[u] = iv[u];
            if (!ok || u >= nv) r[u] = T(0);
        }
        T v4 = __shfl_down(r[0], 1, 64);
        if (gx == gpr - 1) v4 = T(0);
        const T wyz = wz * wy[b];
        s0 += wyz * (wx0[0] * r[0] + wx0[1] * r[1] + wx0[2] * r[2]);
        s1 += wyz * (wx1[0] * r[2] + wx1[1] * r[3] + wx1[2] * v4);
    }
    if (q > 0) {
        sh[w][q - 1][0][lane] = s0;
        sh[w][q - 1][1][lane] = s1;
    }
    __syncthreads();
    if (q > 0 || done) return;
    s0 += sh[w][0][0][lane] + sh[w][1][0][lane];
    s1 += sh[w][0][1][lane] + sh[w][1][1][lane];
    if (own0) rc[e] = dg[0] != T(0) ? s0 : T(0);
    if (own1) rc[e + 1] = dg[1] != T(0) ? s1 : T(0);
    if (F.x1) {
        if (dg[0] != T(0)) F.x1[e] = F.c2 * s0 / dg[0];
        if (dg[1] != T(0)) F.x1[e + 1] = F.c2 * s1 / dg[1];
    }
}

// x(i, j, k) += (P e)(i, j, k) at the regular unknown fine nodes; an irregular node (next
// to the body) keeps x and gets its correction from the post-smoothing.  Interpolating the
// coarse correction there, from coarse nodes that see another interface position, makes the
// cycle amplify errors next to the body (a V-cycle with 3 + 3 steps then grows the error
// 7.6-fold per cycle on 64^3 with 8 spheres; without those corrections it contracts by 0.3).
// Block 64 x 4: lane l of
// wavefront w takes the interior nodes i0 .. i0 + 3 (i0 = 1 + 256 blockIdx.x + 4 l) of row
// j = 1 + 4 blockIdx.y + w in the planes k = 2 blockIdx.z and 2 blockIdx.z + 1 (the interior
// ones), which interpolate from the same two coarse planes.  A fine point i lies in the
// coarse interval starting at min(i / 2, nc - 2) (coarse point I is fine point 2I, the last
// one excepted), so the lane's nodes interpolate from the four coarse x points a0 .. a0 + 3
// of four coarse rows.  Every load is issued at once (4-vectors: x of both planes, the four
// coarse rows, the x weights; vectors and weight tables carry padding past their ends): the
// coarse rows are combined in y, then in z for each plane, then each node interpolates in
// x.  x is stored as one 4-vector where all four nodes are unknowns.
template <typename T>
__global__ void __launch_bounds__(256) k_mg_prolong_add(int nfx, int nfy, int nfz, int ncx, int ncy, int ncz,
                                                        MgAxis<T> ax, MgAxis<T> ay, MgAxis<T> az,
                                                        const uint32_t *__restrict__ skip, int W,
                                                        const T *__restrict__ e, T *__restrict__ x)
{
    using V = typename MgVec4<T>::type;
    // threads take the 4-node groups of a plane's rows in order: no lane idles on short rows (130^3
    // FP32 5.3 us against 7.0 with a row segment per wavefront, 512^3 210 against 219)
    const int gpr = (nfx - 2 + 3) / 4, it = (int)(blockIdx.x * 256 + threadIdx.x), row = it / gpr;
    const int j = 1 + row, kp = 2 * (int)blockIdx.z, i0 = 1 + 4 * (it - row * gpr);
    if (j > nfy - 2) return;
    const int nv = min(4, nfx - 1 - i0);
    const int a0 = min(i0 >> 1, ncx - 2), b = min(j >> 1, ncy - 2), c = min(kp >> 1, ncz - 2);
    const size_t cplane = (size_t)ncx * ncy, fplane = (size_t)nfx * nfy;
    const T *e00 = e + (size_t)c * cplane + (size_t)b * ncx + a0;   // coarse (a0, b, c)
    bool ok[2];
    size_t ef[2];
    V xv[2];
    uint32_t sk[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int k = kp + h;
        ok[h] = k >= 1 && k <= nfz - 2;
        const int kc = ok[h] ? k : 1;
        ef[h] = (size_t)i0 + (size_t)nfx * j + (size_t)kc * fplane;
        xv[h] = *reinterpret_cast<const V *>(x + ef[h]);
        // skip bits (solid and irregular nodes) of nodes i0 .. i0 + 3: words read in pairs,
        // the array carries two words of padding
        const uint32_t *w = skip + ((size_t)kc * nfy + j) * W + (i0 >> 5);
        sk[h] = (uint32_t)((((uint64_t)w[0]) | ((uint64_t)w[1] << 32)) >> (i0 & 31)) & 0xFu;
    }
    const V q00 = *reinterpret_cast<const V *>(e00);
    const V q10 = *reinterpret_cast<const V *>(e00 + ncx);
    const V q01 = *reinterpret_cast<const V *>(e00 + cplane);
    const V q11 = *reinterpret_cast<const V *>(e00 + cplane + ncx);
    const V wxv = *reinterpret_cast<const V *>(ax.pw + i0);
    const T wy = ay.pw[j];
    const T lo[4] = {lerp_(wy, q00.x, q10.x), lerp_(wy, q00.y, q10.y), lerp_(wy, q00.z, q10.z), lerp_(wy, q00.w, q10.w)};
    const T hi[4] = {lerp_(wy, q01.x, q11.x), lerp_(wy, q01.y, q11.y), lerp_(wy, q01.z, q11.z), lerp_(wy, q01.w, q11.w)};
    // (y, on the coarse planes c, c + 1)
    const T wx[4] = {wxv.x, wxv.y, wxv.z, wxv.w};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (!ok[h]) continue;
        const T wz = az.pw[kp + h];
        const T ryz[4] = {lerp_(wz, lo[0], hi[0]), lerp_(wz, lo[1], hi[1]), lerp_(wz, lo[2], hi[2]), lerp_(wz, lo[3], hi[3])};
        T add[4];
        bool m[4];
        bool all = nv == 4;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int d = min((i0 + u) >> 1, ncx - 2) - a0;   // 0 .. 2
            const T l = d == 0 ? ryz[0] : (d == 1 ? ryz[1] : ryz[2]);
            const T r = d == 0 ? ryz[1] : (d == 1 ? ryz[2] : ryz[3]);
            add[u] = lerp_(wx[u], l, r);
            m[u] = u < nv && !((sk[h] >> u) & 1u);   // regular unknowns only (interior, no skip bit)
            all = all && m[u];
        }
        V xo = xv[h];
        if (all) {
            xo.x += add[0];
            xo.y += add[1];
            xo.z += add[2];
            xo.w += add[3];
            *reinterpret_cast<V *>(x + ef[h]) = xo;
        } else {
            const T xs[4] = {xo.x, xo.y, xo.z, xo.w};
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (m[u]) x[ef[h] + u] = xs[u] + add[u];
        }
    }
}

// The coarsest level's Chebyshev-Jacobi iteration on K x = rho from x = 0, all `steps` steps
// in one workgroup (the level has at most MG_LDS_NODES interior nodes): x_k and x_{k+1} live in
// two LDS arrays that swap roles every step, one barrier apart, on the level's grid with its
// walls (0 in every iterate, so a neighbour needs no test).  Each thread keeps, for its nodes
// q = t + MG_LDS_THREADS u (interior, x fastest), x_k, x_{k-1}, the K row and rho divided by
// the row's diagonal (the tables' regular row, or the stored Shortley-Weller row of an
// irregular node) and the LDS places of the row's neighbours in registers.  Nodes that are not
// unknowns stay 0.  x_steps goes to the unknown nodes of out.
//
// A step is bound by its LDS reads (six per node) and the vector instructions beside them; with
// an interior-only array, whose wall neighbours were selected away in every read, the solve of
// 16^3 nodes (8 steps) took 14.8 us in FP32 and 22.3 in FP64, now 13.5 and 17.3.
template <typename T>
__global__ void __launch_bounds__(MG_LDS_THREADS) k_mg_coarsest(int nx, int ny, int nz, Coef<T> cf,
                                                                const int8_t *__restrict__ type,
                                                                const int *__restrict__ irr_map,
                                                                const T *__restrict__ k7, const T *__restrict__ rho,
                                                                T *__restrict__ out, int steps,
                                                                const T *__restrict__ c1, const T *__restrict__ c2,
                                                                const DevState *st)
{
    constexpr int NPT = MG_LDS_NODES / MG_LDS_THREADS;
    __shared__ T xs[2 * MG_LDS_PADDED];
    __shared__ T cs[2 * MG_MAX_COARSE_STEPS];
    const int done = st ? st->done : 0;   // used at the end: nothing waits for it
    const int ni = nx - 2, nj = ny - 2, nk = nz - 2, nij = ni * nj, nint = nij * nk, nxy = nx * ny, nn = nxy * nz;
    const int t = (int)threadIdx.x;
    T ko[NPT][6], rh[NPT], x[NPT], xp[NPT];
    int at[NPT];                          // the node, also its place in LDS
    bool act[NPT];
    // The loads of all nodes are issued at once (one past the level's interior reads node 0),
    // then those of the irregular rows' stored K rows, into registers of their own.
    int8_t ty[NPT];
    int irl[NPT];
    T tab[NPT][7];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
        const int q = t + MG_LDS_THREADS * u, qq = q < nint ? q : 0;
        const int k = qq / nij, r = qq - k * nij, j = r / ni, i = r - j * ni;
        at[u] = (i + 1) + nx * (j + 1) + nxy * (k + 1);
        ty[u] = type[at[u]];
        rh[u] = rho[at[u]];
        irl[u] = irr_map[at[u]];
        const T *cx = cf.c[0] + 8 * (i + 1), *cy = cf.c[1] + 8 * (j + 1), *cz = cf.c[2] + 8 * (k + 1);
        tab[u][0] = cx[6] + cy[6] + cz[6];
        tab[u][1] = cx[5]; tab[u][2] = cx[7];
        tab[u][3] = cy[5]; tab[u][4] = cy[7];
        tab[u][5] = cz[5]; tab[u][6] = cz[7];
        if (q >= nint) ty[u] = 0;
    }
    if (t < steps) {
        cs[t] = c1[t];
        cs[MG_MAX_COARSE_STEPS + t] = c2[t];
    }
    for (int e = t; e < nn; e += MG_LDS_THREADS) {
        xs[e] = T(0);
        xs[MG_LDS_PADDED + e] = T(0);
    }
    // as many nodes' rows in flight as the registers hold
    constexpr int ROWS = sizeof(T) == 4 ? NPT : 2;
#pragma unroll
    for (int u0 = 0; u0 < NPT; u0 += ROWS) {
        T row[ROWS][7];
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (ty[u0 + r] == 2) {
                const T *p = k7 + 7 * (size_t)irl[u0 + r];
#pragma unroll
                for (int v = 0; v < 7; ++v) row[r][v] = p[v];
            }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int u = u0 + r;
            const bool irr = ty[u] == 2;
            act[u] = irr || ty[u] == 1;
            // rows scaled by 1 / diag K: (rho - K x) / diag = rho' - x - sum_v ko'_v x_v
            const T rd = T(1) / (act[u] ? (irr ? row[r][0] : tab[u][0]) : T(1));
            rh[u] = act[u] ? rh[u] * rd : T(0);
#pragma unroll
            for (int v = 0; v < 6; ++v) ko[u][v] = act[u] ? (irr ? row[r][1 + v] : tab[u][1 + v]) * rd : T(0);
            x[u] = T(0);
            xp[u] = T(0);
        }
    }
    __syncthreads();
    // step s reads x_s from one array and writes x_{s+1} into the other (nodes that are not
    // unknowns stay 0 in both), so one barrier per step separates them
    auto step = [&](const T *cur, T *nxt, int s) __attribute__((always_inline)) {
        const T a1 = cs[s], a2 = cs[MG_MAX_COARSE_STEPS + s];
#pragma unroll
        for (int u = 0; u < NPT; ++u) {
            const T *c = cur + at[u];
            T kx = x[u];
            kx += ko[u][0] * c[-1];
            kx += ko[u][1] * c[1];
            kx += ko[u][2] * c[-nx];
            kx += ko[u][3] * c[nx];
            kx += ko[u][4] * c[-nxy];
            kx += ko[u][5] * c[nxy];
            const T xn = x[u] + a1 * (x[u] - xp[u]) + a2 * (rh[u] - kx);
            xp[u] = x[u];
            if (act[u]) {
                nxt[at[u]] = xn;
                x[u] = xn;
            }
        }
        __syncthreads();
    };
    int s = 0;
    for (; s + 1 < steps; s += 2) {
        step(xs, xs + MG_LDS_PADDED, s);
        step(xs + MG_LDS_PADDED, xs, s + 1);
    }
    if (s < steps) step(xs, xs + MG_LDS_PADDED, s);
    if (done) return;
#pragma unroll
    for (int u = 0; u < NPT; ++u)
        if (act[u]) out[at[u]] = x[u];
}

// The value of the lane before / after within 16 lanes (0 beyond them).
__device__ __forceinline__ float lane_before(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_after(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x101, 0xf, 0xf, true));
}
template <typename F>
__device__ __forceinline__ double both_halves(double v, F f)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__float_as_int(f(__int_as_float((int)(b & 0xffffffffll))));
    const uint32_t hi = (uint32_t)__float_as_int(f(__int_as_float((int)(b >> 32))));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double lane_before(double v)
{
    return both_halves(v, [](float h) { return lane_before(h); });
}
__device__ __forceinline__ double lane_after(double v)
{
    return both_halves(v, [](float h) { return lane_after(h); });
}

// The same iteration on a level of at most 16 interior nodes per axis (every cube's coarsest
// level): 16 lanes take a row of x, a thread four nodes along z, z fastest in LDS.  The x
// neighbours come from the adjacent lanes' registers, three quarters of the z neighbours from the
// thread's own, and the y neighbours of all four nodes in one read: 5 LDS instructions a step
// instead of 28 (FP32), and a third of the loads before the steps.  Lanes, rows and planes past
// the interior hold 0.  Solve of 16^3 nodes, 8 steps (us): FP32 8.6 against 13.1,
// FP64 11.2 against 16.6.
constexpr int MG_C16 = 16;
template <typename T>
__global__ void __launch_bounds__(MG_LDS_THREADS) k_mg_coarsest16(int nx, int ny, int nz, Coef<T> cf,
                                                                  const int8_t *__restrict__ type,
                                                                  const int *__restrict__ irr_map,
                                                                  const T *__restrict__ k7, const T *__restrict__ rho,
                                                                  T *__restrict__ out, int steps,
                                                                  const T *__restrict__ c1, const T *__restrict__ c2,
                                                                  const DevState *st)
{
    // z column of LDS: KO places before k = 0 (so that four nodes start at 16 bytes), a pitch that
    // spreads 8 lanes' 16-byte reads over all banks
    constexpr int KO = 16 / (int)sizeof(T), LZ = sizeof(T) == 4 ? 24 : 22, LY = LZ * MG_C16;
    struct alignas(16) Four {
        T v[4];
    };
    __shared__ alignas(16) T xs[2][(MG_C16 + 2) * LY];
    __shared__ T cs[2 * MG_MAX_COARSE_STEPS];
    const int done = st ? st->done : 0;   // used at the end: nothing waits for it
    const int t = (int)threadIdx.x, wv = t >> 6, i = t & 15, j = 4 * (wv & 3) + ((t >> 4) & 3), k0 = 4 * (wv >> 2);
    const int ni = nx - 2, nj = ny - 2, nk = nz - 2, nxy = nx * ny;
    const bool col = i < ni && j < nj;
    const int ic = min(i, ni - 1) + 1, jc = min(j, nj - 1) + 1;
    // all nodes' loads at once, then those of the irregular rows' stored K rows
    int node[4], irl[4];
    int8_t ty[4];
    T rh[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int kc = min(k0 + u, nk - 1) + 1;
        node[u] = ic + nx * jc + nxy * kc;
        ty[u] = type[node[u]];
        rh[u] = rho[node[u]];
        irl[u] = irr_map[node[u]];
    }
    const T *cx = cf.c[0] + 8 * ic, *cy = cf.c[1] + 8 * jc;
    const T kx5 = cx[5], kx6 = cx[6], kx7 = cx[7], ky5 = cy[5], ky6 = cy[6], ky7 = cy[7];
    if (t < steps) {
        cs[t] = c1[t];
        cs[MG_MAX_COARSE_STEPS + t] = c2[t];
    }
    {
        Four *z = reinterpret_cast<Four *>(xs);
        for (int q = t; q < 2 * (MG_C16 + 2) * LY / 4; q += MG_LDS_THREADS) z[q] = Four{{T(0), T(0), T(0), T(0)}};
    }
    T ko[4][6], x[4], xp[4];
    bool act[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int kc = min(k0 + u, nk - 1) + 1;
        const T *cz = cf.c[2] + 8 * kc;
        T row[7] = {kx6 + ky6 + cz[6], kx5, kx7, ky5, ky7, cz[5], cz[7]};
        const bool in = col && k0 + u < nk, irr = in && ty[u] == 2;
        if (irr) {
            const T *p = k7 + 7 * (size_t)irl[u];
#pragma unroll
            for (int v = 0; v < 7; ++v) row[v] = p[v];
        }
        act[u] = irr || (in && ty[u] == 1);
        // rows scaled by 1 / diag K: (rho - K x) / diag = rho' - x - sum_v ko'_v x_v
        const T rd = act[u] ? T(1) / row[0] : T(0);
        rh[u] *= rd;
#pragma unroll
        for (int v = 0; v < 6; ++v) ko[u][v] = row[1 + v] * rd;
        if (!act[u]) rh[u] = T(0);
        x[u] = T(0);
        xp[u] = T(0);
    }
    const int at = (j + 1) * LY + i * LZ + KO + k0;
    __syncthreads();
    auto step = [&](const T *cur, T *nxt, int s) __attribute__((always_inline)) {
        const T a1 = cs[s], a2 = cs[MG_MAX_COARSE_STEPS + s];
        const Four lo = *reinterpret_cast<const Four *>(cur + at - LY), hi = *reinterpret_cast<const Four *>(cur + at + LY);
        const T zlo = cur[at - 1], zhi = cur[at + 4];
        Four xn;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            T kx = x[u];
            kx += ko[u][0] * lane_before(x[u]);
            kx += ko[u][1] * lane_after(x[u]);
            kx += ko[u][2] * lo.v[u];
            kx += ko[u][3] * hi.v[u];
            kx += ko[u][4] * (u == 0 ? zlo : x[u == 0 ? 0 : u - 1]);
            kx += ko[u][5] * (u == 3 ? zhi : x[u == 3 ? 3 : u + 1]);
            xn.v[u] = x[u] + a1 * (x[u] - xp[u]) + a2 * (rh[u] - kx);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            xp[u] = x[u];
            x[u] = act[u] ? xn.v[u] : T(0);
            xn.v[u] = x[u];
        }
        *reinterpret_cast<Four *>(nxt + at) = xn;
        __syncthreads();
    };
    int s = 0;
    for (; s + 1 < steps; s += 2) {
        step(xs[0], xs[1], s);
        step(xs[1], xs[0], s + 1);
    }
    if (s < steps) step(xs[0], xs[1], s);
    if (done) return;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (act[u]) out[node[u]] = x[u];
}

// Temporally blocked Chebyshev-Jacobi steps on a coarse level (launch_mg_smooth_tb).  The
// block owns a tile of MG_TB_TS^3 nodes.  x_0 is loaded on the tile and H layers around it
// (edge E, 0 at nodes that are not unknowns and outside the grid's interior) into LDS; the
// steps run on the tile and H - 1 layers (edge G), whose K row, rho and x_{k-1} the points'
// threads hold in registers.  Every step updates all of those points: after s steps the
// points within H - s layers of the tile hold exactly the values of s single sweeps (the
// others have read stale neighbours, which move inwards one layer per step).  H is the least
// that the pass needs: the steps, and one layer more for the residual on the tile, two for its
// restriction.  x_k and x_{k+1} live in two LDS arrays that swap roles, one barrier per step.
// The arithmetic is that of the single sweep (row7, cheb_next), bit for bit k_sweep_short's.
//
// The levels this runs on are bound by latency: the kernel waits for memory twice (all loads
// that depend on indices only, then the irregular nodes' stored K rows into registers of
// their own) and for its steps.  (The FP64 form with four layers and the coarse correction, which
// four smoothing steps take, spills 40 registers: 100^3 V-cycle 249 us against 342 with the passes
// before.)  With four layers for every pass, each point's row loaded
// inside its type branch (a round trip per point) and the solver's state read first, a pass
// took 9.3 (before the coarse correction) and 11.5 us (after it) in FP32, 15.4 and 18.0 in
// FP64 (66^3 and 34^3 levels, averages); now 7.5, 7.3, 13.3 and 11.4.
//
// What a pass writes besides x on its tile: nothing (TB_X), the residual on the tile (TB_RES),
// or the residual restricted into the next coarser level (TB_RESTRICT: that level's rho and
// first step, as k_mg_restrict forms them, for the coarse nodes whose centre lies in the tile).
// With PRO the pass starts from x + P e at the regular unknowns (the coarse correction added on
// load, as k_mg_prolong_add forms it) instead of x.
enum { TB_X = 0, TB_RES = 1, TB_RESTRICT = 2 };

template <typename T, int OUT, bool PRO, int H>
__global__ void __launch_bounds__(MG_TB_THREADS) k_mg_smooth_tb(int nx, int ny, int nz, Coef<T> cf,
                                                                const int8_t *__restrict__ type,
                                                                const int *__restrict__ irr_map,
                                                                const T *__restrict__ k7, const T *__restrict__ rho,
                                                                const T *__restrict__ xin, T *__restrict__ xout,
                                                                T *__restrict__ rout, MgSteps<T> S, const DevState *st,
                                                                MgTransfer<T> tr, const T *__restrict__ ec,
                                                                T *__restrict__ rc, MgFirst<T> F)
{
    constexpr int TS = MG_TB_TS, NTH = MG_TB_THREADS, E = TS + 2 * H, E2 = E * E, E3 = E2 * E, G = E - 2, G3 = G * G * G;
    constexpr int NX = (E3 + NTH - 1) / NTH, NG = (G3 + NTH - 1) / NTH;   // points per thread: loaded, stepped
    constexpr int RE = TS + 1;                            // residual edge: the tile and the layer above it
    static_assert(TS % 2 == 0, "a tile holds whole coarse cells");
    __shared__ T xs[2][E3];
    __shared__ T rs[OUT == TB_RESTRICT ? RE * RE * RE : 1];
    const int done = st ? st->done : 0;   // used before the first store: nothing waits for it
    const int t = (int)threadIdx.x;
    // first node of the extended tile
    const int o[3] = {1 + TS * (int)blockIdx.x - H, 1 + TS * (int)blockIdx.y - H, 1 + TS * (int)blockIdx.z - H};
    // TB_RESTRICT: thread t < (TS/2)^3 restricts into coarse node (I, J, K) = (1 + TS/2 b + c)
    // at the end
    constexpr int CT = TS / 2, CT3 = CT * CT * CT;
    const int ci = t % CT, cj = (t / CT) % CT, ck = t / (CT * CT);
    const int cI = 1 + CT * (int)blockIdx.x + ci, cJ = 1 + CT * (int)blockIdx.y + cj, cK = 1 + CT * (int)blockIdx.z + ck;
    const bool cown = OUT == TB_RESTRICT && t < CT3 && cI <= tr.nc[0] - 2 && cJ <= tr.nc[1] - 2 && cK <= tr.nc[2] - 2;
    const size_t ce = cown ? (size_t)cI + (size_t)tr.nc[0] * (cJ + (size_t)tr.nc[1] * cK) : 0;
    auto inside = [&](int i, int j, int k) {
        return i >= 1 && i <= nx - 2 && j >= 1 && j <= ny - 2 && k >= 1 && k <= nz - 2;
    };
    auto node = [&](int i, int j, int k) { return (size_t)i + (size_t)nx * ((size_t)j + (size_t)ny * k); };
    // ---- loads that depend on indices only, all in flight together (points outside the grid's
    // interior read node 0 and clamped table entries)
    T x0[NX], pe[NX];
    bool xin_ok[NX];
    int8_t xty[NX];
#pragma unroll
    for (int u = 0; u < NX; ++u) {
        const int q = min(t + NTH * u, E3 - 1);
        const int i = o[0] + q % E, j = o[1] + (q / E) % E, k = o[2] + q / E2;
        xin_ok[u] = inside(i, j, k);
        const size_t e = xin_ok[u] ? node(i, j, k) : 0;
        x0[u] = xin[e];
        pe[u] = T(0);
        xty[u] = 0;
        if (PRO) {
            // (P e)(i, j, k): the coarse interval of each index, combined in y, then z, then x
            const int ic = min(max(i, 1), nx - 2), jc = min(max(j, 1), ny - 2), kc = min(max(k, 1), nz - 2);
            const int ncx = tr.nc[0], ncy = tr.nc[1], ncz = tr.nc[2];
            const int a0 = min(ic >> 1, ncx - 2), b0 = min(jc >> 1, ncy - 2), c0 = min(kc >> 1, ncz - 2);
            const size_t cpl = (size_t)ncx * ncy;
            const T *e00 = ec + (size_t)c0 * cpl + (size_t)b0 * ncx + a0;
            const T wx = tr.ax[0].pw[ic], wy = tr.ax[1].pw[jc], wz = tr.ax[2].pw[kc];
            xty[u] = type[e];
            T ryz[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const T lo = lerp_(wy, e00[h], e00[ncx + h]), hi = lerp_(wy, e00[cpl + h], e00[cpl + ncx + h]);
                ryz[h] = lerp_(wz, lo, hi);
            }
            pe[u] = lerp_(wx, ryz[0], ryz[1]);
        }
    }
    T rh[NG], kd[NG], ko[NG][6], xp[NG];
    int8_t ty[NG];
    int irl[NG];
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const int g = min(t + NTH * u, G3 - 1);
        const int i = o[0] + 1 + g % G, j = o[1] + 1 + (g / G) % G, k = o[2] + 1 + g / (G * G);
        const bool in = t + NTH * u < G3 && inside(i, j, k);
        const size_t e = in ? node(i, j, k) : 0;
        ty[u] = type[e];
        rh[u] = rho[e];
        irl[u] = irr_map[e];
        if (!in) ty[u] = 0;
        const int ic = min(max(i, 1), nx - 2), jc = min(max(j, 1), ny - 2), kc = min(max(k, 1), nz - 2);
        const T *cx = cf.xs + (size_t)5 * cf.xp + ic, *cy = cf.c[1] + 8 * jc, *cz = cf.c[2] + 8 * kc;
        kd[u] = (cx[cf.xp] + cy[6]) + cz[6];
        ko[u][0] = cx[0]; ko[u][1] = cx[2 * cf.xp];
        ko[u][2] = cy[5]; ko[u][3] = cy[7];
        ko[u][4] = cz[5]; ko[u][5] = cz[7];
        xp[u] = T(0);
    }
    T cw[10];                              // TB_RESTRICT: the coarse node's nine weights and diagonal
    if (OUT == TB_RESTRICT) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            cw[c] = tr.ax[0].rw[cown ? 3 * cI + c : 0];
            cw[3 + c] = tr.ax[1].rw[cown ? 3 * cJ + c : 0];
            cw[6 + c] = tr.ax[2].rw[cown ? 3 * cK + c : 0];
        }
        cw[9] = F.diag[ce];
    }
    // ---- the irregular nodes' stored K rows
    T row[NG][7];
#pragma unroll
    for (int u = 0; u < NG; ++u)
        if (ty[u] == 2) {
            const T *r = k7 + 7 * (size_t)irl[u];
#pragma unroll
            for (int v = 0; v < 7; ++v) row[u][v] = r[v];
        }
#pragma unroll
    for (int u = 0; u < NX; ++u) {
        const int q = t + NTH * u;
        T v = xin_ok[u] ? x0[u] : T(0);
        if (PRO && xin_ok[u] && xty[u] == 1) v = v + pe[u];
        if (q < E3) xs[0][q] = v;
    }
    bool act[NG];
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const bool irr = ty[u] == 2;
        act[u] = irr || ty[u] == 1;
        kd[u] = act[u] ? (irr ? row[u][0] : kd[u]) : T(1);
#pragma unroll
        for (int v = 0; v < 6; ++v) ko[u][v] = act[u] ? (irr ? row[u][1 + v] : ko[u][v]) : T(0);
        rh[u] = act[u] ? rh[u] : T(0);
    }
    __syncthreads();
    // point u of the thread in the extended tile
    auto at_of = [&](int u) {
        const int g = min(t + NTH * u, G3 - 1);
        return (1 + g % G) + E * (1 + (g / G) % G) + E2 * (1 + g / (G * G));
    };
    const T *cur = xs[0];
    auto kx_of = [&](int u, int q, T x) {
        return row7(kd[u], x, ko[u][0], cur[q - 1], ko[u][1], cur[q + 1], ko[u][2], cur[q - E], ko[u][3], cur[q + E],
                    ko[u][4], cur[q - E2], ko[u][5], cur[q + E2]);
    };
    for (int s = 0; s < S.n; ++s) {
        const T c1 = S.c1[s], c2 = S.c2[s];
        T *nxt = xs[(s + 1) & 1];
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            const int q = at_of(u);
            const T x = cur[q];
            const T kx = kx_of(u, q, x);
            const T xn = act[u] ? cheb_next(x, xp[u], c1, c2, rh[u] - kx, kd[u]) : T(0);
            xp[u] = x;
            if (t + NTH * u < G3) nxt[q] = xn;
        }
        __syncthreads();
        cur = nxt;
    }
    if (done) return;
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const int q = at_of(u), ii = q % E, jj = (q / E) % E, kk = q / E2;
        if (t + NTH * u >= G3) continue;
        const int lo = min(min(ii, jj), kk) - H, hi = max(max(ii, jj), kk) - H;   // tile: 0 .. TS - 1
        const T x = cur[q];
        if (OUT == TB_RESTRICT && lo >= 0 && hi <= TS)
            rs[(ii - H) + RE * ((jj - H) + RE * (kk - H))] = act[u] ? rh[u] - kx_of(u, q, x) : T(0);
        if (!act[u] || lo < 0 || hi >= TS) continue;
        const size_t e = node(o[0] + ii, o[1] + jj, o[2] + kk);
        xout[e] = x;
        if (OUT == TB_RES) rout[e] = rh[u] - kx_of(u, q, x);
    }
    if (OUT == TB_RESTRICT) {
        // coarse node (I, J, K): its fine points 2I - 1 .. 2I + 1 are the points 2c .. 2c + 2 of
        // the tile (and the layer above it) in each direction
        __syncthreads();
        if (cown) {
            T acc = T(0);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    const T wyz = cw[6 + c] * cw[3 + b];
                    const T *r = rs + (2 * ck + c) * RE * RE + (2 * cj + b) * RE + 2 * ci;
                    acc += wyz * (cw[0] * r[0] + cw[1] * r[1] + cw[2] * r[2]);
                }
            }
            const T cdg = cw[9];
            rc[ce] = cdg != T(0) ? acc : T(0);
            if (F.x1 && cdg != T(0)) F.x1[ce] = F.c2 * acc / cdg;
        }
    }
}

// diag[e] = the diagonal of K at node e if it is an unknown (the 1D tables of a regular node,
// summed as cx + (cy + cz), or the stored row of an irregular one), 0 otherwise
template <typename T>
__global__ void k_mg_diag(int nx, int ny, int nz, Coef<T> cf, const int8_t *__restrict__ type,
                          const int *__restrict__ irr_map, const T *__restrict__ k7, T *__restrict__ diag)
{
    const size_t n = (size_t)nx * ny * nz;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(e % nx), j = (int)((e / nx) % ny), k = (int)(e / ((size_t)nx * ny));
        const int8_t t = type[e];
        T d = T(0);
        if (t == 1) d = cf.c[0][8 * i + 6] + (cf.c[1][8 * j + 6] + cf.c[2][8 * k + 6]);
        else if (t == 2) d = k7[7 * (size_t)irr_map[e]];
        diag[e] = d;
    }
}

// map[node] = irregular row of the node (the rows list nodes in increasing order)
__global__ void k_mg_irr_map(int nirr, const int *__restrict__ nodes, int *__restrict__ map)
{
    const int r = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (r < nirr) map[nodes[r]] = r;
}

}  // namespace

template <typename T>
void launch_mg_diag(hipStream_t s, int nx, int ny, int nz, const Coef<T> &cf, const int8_t *type, const int *irr_map,
                    const T *k7, T *diag)
{
    const size_t n = (size_t)nx * ny * nz;
    k_mg_diag<T><<<(unsigned)std::min<size_t>((n + 255) / 256, 4096), 256, 0, s>>>(nx, ny, nz, cf, type, irr_map, k7,
                                                                                  diag);
}

template <typename T>
void launch_mg_restrict(hipStream_t s, const MgTransfer<T> &t, const T *r, T *rc, const MgFirst<T> &first)
{
    dim3 grid((unsigned)((t.nc[0] - 2 + 127) / 128), (unsigned)((t.nc[1] - 2 + 3) / 4), (unsigned)(t.nc[2] - 2));
    k_mg_restrict<T><<<grid, dim3(64, 4), 0, s>>>(t.nc[0], t.nc[1], t.nf[0], t.nf[1], t.ax[0], t.ax[1], t.ax[2], r,
                                                  rc, first);
}

// Tiles of a kernel whose blocks march over tiles_x x tiles_y columns of nzi planes.  The march is
// bound by the latency of its plane steps: all blocks run in one round, as many as fit on the current
// device at once (z-chunks of at least min_tz planes).
static Tiling march_tiling(const void *fn, int threads, int tiles_x, int tiles_y, int nzi, int min_tz = 2)
{
    int per_cu = 0, dev = 0, ncu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
        ncu = 256;
    Tiling tl{};
    tl.tiles_x = tiles_x;
    tl.tiles_y = tiles_y;
    const int per_plane = tiles_x * tiles_y, want = std::max(1, per_cu * ncu / per_plane);
    tl.TZ = std::max(std::min(min_tz, nzi), (nzi + want - 1) / want);
    tl.zchunks = (nzi + tl.TZ - 1) / tl.TZ;
    tl.ntiles = per_plane * tl.zchunks;
    tl.nblk = (tl.ntiles + NXCD - 1) / NXCD * NXCD;
    return tl;
}

// Which grids restrict with the short kernel: up to RRS_MAX_BYTES per vector.  Its twice-formed rows
// and planes lose where the march has planes enough to overlap.  Measured (us, short against
// march): FP32 66^3 5.6 / 11.2, 82^3 8.3 / 8.8, 98^3 (3.5 MB) 8.5 / 8.6, 130^3 16.5 / 11.3; FP64 32^3
// 6.6 / 13.7, 70^3 (2.5 MB) 7.5 / 10.7, 82^3 (4.1 MB) 11.7 / 10.7, 211x147x99 31 / 20.
constexpr size_t RRS_MAX_BYTES = 3300000;
template <typename T>
static bool resid_restrict_short(const Geom &g)
{
    return (size_t)(g.nx - 2) * (g.ny - 2) * (g.nz - 2) * sizeof(T) <= RRS_MAX_BYTES;
}

// the marching kernel of a grid: the fifth-node path (more registers) only where some lane 63 owns
// its second coarse node (128) and that node's last fine point (257) is interior; with an odd nx that
// is so from nx = 259, where one segment still covers the coarse row
static bool rr_fifth(const Geom &g) { return g.nx - 2 >= 257; }
static bool rr_half(const Geom &g) { return g.nx - 2 <= 128; }
template <typename T>
static auto rr_kernel(const Geom &g)
{
    return rr_fifth(g) ? &k_mg_resid_restrict<T, true, false>
           : rr_half(g) ? &k_mg_resid_restrict<T, false, true>
                        : &k_mg_resid_restrict<T, false, false>;
}

template <typename T>
void launch_mg_resid_restrict(hipStream_t s, const Geom &g, const Tiling &tl, const Coef<T> &cf, const uint32_t *skip,
                              const T *x, const T *rho, const T *ri, const MgTransfer<T> &t, T *rc,
                              const MgFirst<T> &first, const DevState *st)
{
    if (resid_restrict_short<T>(g)) {
        const int gpr = (g.nx - 2 + 3) / 4;
        const int nbx = (gpr * (t.nc[1] - 2) + RRS_WAVE * RRS_WAVES - 1) / (RRS_WAVE * RRS_WAVES);
        const int nb = (nbx * (t.nc[2] - 2) + NXCD - 1) / NXCD * NXCD;
        k_mg_resid_restrict_short<T><<<nb, dim3(64, 3, RRS_WAVES), 0, s>>>(g, cf, skip, x, rho, ri, t.nc[0], t.nc[1],
                                                                          t.nc[2], t.ax[0], t.ax[1], t.ax[2], gpr, nbx,
                                                                          rc, first, st);
        return;
    }
    rr_kernel<T>(g)<<<tl.nblk, dim3(64, RR_ROWS + 1), 0, s>>>(g, tl, cf, skip, x, rho, ri, t.nc[0], t.nc[1], t.nc[2],
                                                              t.ax[0], t.ax[1], t.ax[2], rc, first, st);
}

// Which grids take these marches: those with more than MARCH_MIN_BYTES per vector; where the sweeps
// would be short ones (up to 65 MB), only with at least MARCH_MIN_FILL of the lanes on the rows: a
// wavefront takes 256 nodes of a row, and the short sweeps idle none.  On smaller grids the sweeps run
// from the Infinity Cache and their launches cost less than the marches' few wavefronts.  Measured
// (6 iterations of a solve in ms, marches against sweeps): FP32 cubes 180^3 (23 MB) 2.89 / 2.87, 202^3
// 3.41 / 3.46, 220^3 (42 MB) 4.01 / 4.12, 245^3 4.99 / 5.28; lanes in use at 43 to 49 MB: 400x180x180 (0.78)
// 4.99 / 4.95, 520x150x150 (0.67) 4.72 / 4.59, 150x280x280 (0.58) 4.75 / 4.64, 102x340x340 (0.39) 5.49 /
// 5.03, 34x600x600 (0.13) 9.76 / 6.95; beyond 65 MB 130x370x370 (0.50) 6.99 / 7.69, 34x740x740 14.3 / 14.9.
// FP64 162^3 (33 MB) 3.68 / 3.68, 175^3 (42 MB, 0.68) 4.24 / 4.25, 190^3 (0.73) 4.86 / 5.00, 130x200x200
// (0.50) 4.42 / 4.25, 66x300x300 (0.25) 6.43 / 5.25; beyond 65 MB 130x260x260 6.43 / 7.33.  The FP64 pair
// with the edge nodes of rows beyond 256 interior nodes spills its registers (300^3: 717 us against
// 242 + 294), so those grids sweep twice.
constexpr size_t MARCH_MIN_BYTES = 40000000;
constexpr double MARCH_MIN_FILL = 0.7;
// The marches multiply by 1 / diag K (recip), which has to be a normal number: in FP32 the
// reciprocal of a diagonal beyond 2^126 (a spacing below 2.6e-19) is flushed to 0, and that of one
// below 2^-126 is infinite, where the sweeps' division still gives the step.  A hundred binary
// digits either way are far from both ends.
template <typename T>
static bool reciprocals_normal(const Geom &g)
{
    constexpr double big = sizeof(T) == 4 ? 0x1p100 : 0x1p1000;
    return g.kd_max < big && g.kd_min > 1.0 / big;
}
template <typename T>
bool mg_second_pays(const Geom &g)
{
    const int segs = (g.nx - 2 + 255) / 256;
    return (size_t)(g.nx - 2) * (g.ny - 2) * (g.nz - 2) * sizeof(T) > MARCH_MIN_BYTES && reciprocals_normal<T>(g) &&
           (!sweeps_short<T>(g) || g.nx - 2 >= MARCH_MIN_FILL * 256 * segs);
}
template <typename T>
bool mg_pair_pays(const Geom &g)
{
    return mg_second_pays<T>(g) && (sizeof(T) == 4 || g.nx - 2 <= 256);
}

// a launch that stamps the events ev[0], ev[1] (ev non-null) with the kernel's start and end
template <typename... Args>
static void timed_launch(const hipEvent_t *ev, void (*kernel)(Args...), dim3 grid, dim3 block, hipStream_t s, Args... args)
{
    if (ev) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev[0], ev[1], 0, args...);
    else kernel<<<grid, block, 0, s>>>(args...);
}

// the kernels of a grid: more than one segment per row (SEG) or not; the FP64 pair has none of the
// former (mg_pair_pays)
template <typename T>
static auto pair_kernel(const Geom &g)
{
    if constexpr (sizeof(T) == 4) return g.nx - 2 > 256 ? &k_mg_pair<T, true> : &k_mg_pair<T, false>;
    else return &k_mg_pair<T, false>;
}
template <typename T>
static auto second_kernel(const Geom &g)
{
    return g.nx - 2 > 256 ? &k_mg_second<T, true> : &k_mg_second<T, false>;
}

template <typename T>
MgMarches mg_marches(const Geom &g, const MgTransfer<T> &t)
{
    MgMarches m;
    const int segs = (g.nx - 2 + 255) / 256;
    const auto tiling = [&](auto kernel, int waves, int rows) {
        return march_tiling(reinterpret_cast<const void *>(kernel), 64 * waves, segs, (g.ny - 2 + rows - 1) / rows, g.nz - 2);
    };
    if (!resid_restrict_short<T>(g)) {
        const bool half = rr_half(g);
        const int rows = half ? 2 * RR_ROWS + 1 : RR_ROWS;
        m.rr = march_tiling(reinterpret_cast<const void *>(rr_kernel<T>(g)), 64 * (RR_ROWS + 1), (t.nc[0] - 2 + 127) / 128,
                            (t.nc[1] - 2 + rows - 1) / rows, t.nc[2] - 2, half ? 1 : 2);
    }
    if (mg_second_pays<T>(g)) m.second = tiling(second_kernel<T>(g), Second<T>::waves, Second<T>::rows);
    if (mg_pair_pays<T>(g)) m.pair = tiling(pair_kernel<T>(g), Pair<T>::waves, Pair<T>::rows);
    m.set = true;
    return m;
}

template <typename T>
void launch_mg_pair(const Launch &L, const Tiling &tl, const Coef<T> &cf, const Irr<T> &ir, const T *x, const T *rho,
                    T *yi, T *out, double c2a, double c1, double c2, const DevState *st, const hipEvent_t *ev)
{
    const Geom &g = L.g;
    if (ir.n > 0)
        timed_launch(ev ? ev + 2 : nullptr, k_mg_pair_irregular<T>, dim3((8 * ir.n + NT - 1) / NT), dim3(NT), L.stream, g, cf,
                     ir, L.skip, x, rho, yi, out, (T)c2a, (T)c1, (T)c2, st);
    timed_launch(ev, pair_kernel<T>(g), dim3(tl.nblk), dim3(64, Pair<T>::waves), L.stream, g, tl, cf, L.skip, x, rho,
                 (const T *)yi, out, (T)c2a, (T)c1, (T)c2, st);
}

template <typename T>
void launch_mg_second(const Launch &L, const Tiling &tl, const Coef<T> &cf, const Irr<T> &ir, const T *x1, const T *rho,
                      T *out, double c2a, double c1, double c2, const DevState *st, const hipEvent_t *ev)
{
    constexpr int NTH = 64 * Second<T>::waves;
    const int nb = tl.nblk + (8 * ir.n + NTH - 1) / NTH;
    timed_launch(ev, second_kernel<T>(L.g), dim3(nb), dim3(64, Second<T>::waves), L.stream, L.g, tl, cf, ir, L.skip, x1,
                 rho, out, (T)c2a, (T)c1, (T)c2, st);
}

template <typename T>
void launch_mg_prolong_add(hipStream_t s, const MgTransfer<T> &t, const uint32_t *skip_f, int W, const T *e, T *x)
{
    // blockIdx.z = p covers fine planes 2p and 2p + 1 (interior planes 1 .. nf[2] - 2)
    const int groups = (t.nf[0] - 2 + 3) / 4 * (t.nf[1] - 2);
    dim3 grid((unsigned)((groups + 255) / 256), 1, (unsigned)((t.nf[2] - 2) / 2 + 1));
    k_mg_prolong_add<T><<<grid, 256, 0, s>>>(t.nf[0], t.nf[1], t.nf[2], t.nc[0], t.nc[1], t.nc[2], t.ax[0],
                                                     t.ax[1], t.ax[2], skip_f, W, e, x);
}

template <typename T>
void launch_mg_coarsest(hipStream_t s, int nx, int ny, int nz, const Coef<T> &cf, const int8_t *type,
                        const int *irr_map, const T *k7, const T *rho, T *out, int steps, const T *c1, const T *c2,
                        const DevState *st)
{
    // at most 16 interior nodes per axis: a thread's z column and its x row fit the layout
    // (k_mg_coarsest16 has both times)
    if (std::max(nx, std::max(ny, nz)) - 2 <= MG_C16)
        k_mg_coarsest16<T><<<1, MG_LDS_THREADS, 0, s>>>(nx, ny, nz, cf, type, irr_map, k7, rho, out, steps, c1, c2, st);
    else
        k_mg_coarsest<T><<<1, MG_LDS_THREADS, 0, s>>>(nx, ny, nz, cf, type, irr_map, k7, rho, out, steps, c1, c2, st);
}

template <typename T>
void launch_mg_smooth_tb(hipStream_t s, int nx, int ny, int nz, const Coef<T> &cf, const int8_t *type,
                         const int *irr_map, const T *k7, const T *rho, const T *xin, T *xout, T *rout,
                         const MgSteps<T> &S, const DevState *st, const MgTransfer<T> *tr, const T *e_add, T *rc,
                         const MgFirst<T> *first)
{
    const dim3 grid((unsigned)((nx - 2 + MG_TB_TS - 1) / MG_TB_TS), (unsigned)((ny - 2 + MG_TB_TS - 1) / MG_TB_TS),
                    (unsigned)((nz - 2 + MG_TB_TS - 1) / MG_TB_TS));
    const MgTransfer<T> t = tr ? *tr : MgTransfer<T>{};
    const MgFirst<T> F = first ? *first : MgFirst<T>{};
#define CPS_TB_LAUNCH(OUT, PRO, H)                                                                                     \
    k_mg_smooth_tb<T, OUT, PRO, H><<<grid, MG_TB_THREADS, 0, s>>>(nx, ny, nz, cf, type, irr_map, k7, rho, xin, xout,   \
                                                                  rout, S, st, t, e_add, rc, F)
    // the least layers that hold the steps and the residual's (two for its restriction)
#define CPS_TB_LAYERS(OUT, PRO, h)                                                                                     \
    do {                                                                                                               \
        if ((h) <= 2) CPS_TB_LAUNCH(OUT, PRO, 2);                                                                      \
        else if ((h) == 3) CPS_TB_LAUNCH(OUT, PRO, 3);                                                                 \
        else CPS_TB_LAUNCH(OUT, PRO, 4);                                                                               \
    } while (0)
    if (rc) CPS_TB_LAYERS(TB_RESTRICT, false, S.n + 2);
    else if (rout) CPS_TB_LAYERS(TB_RES, false, S.n + 1);
    else if (e_add) CPS_TB_LAYERS(TB_X, true, S.n);
    else CPS_TB_LAYERS(TB_X, false, S.n);
#undef CPS_TB_LAYERS
#undef CPS_TB_LAUNCH
}

void launch_mg_irr_map(hipStream_t s, int nirr, const int *nodes, int *map)
{
    if (nirr > 0) k_mg_irr_map<<<(nirr + 255) / 256, 256, 0, s>>>(nirr, nodes, map);
}

template void launch_mg_coarsest<double>(hipStream_t, int, int, int, const Coef<double> &, const int8_t *, const int *,
                                         const double *, const double *, double *, int, const double *, const double *,
                                         const DevState *);
template void launch_mg_coarsest<float>(hipStream_t, int, int, int, const Coef<float> &, const int8_t *, const int *,
                                        const float *, const float *, float *, int, const float *, const float *,
                                        const DevState *);
template void launch_mg_smooth_tb<double>(hipStream_t, int, int, int, const Coef<double> &, const int8_t *,
                                          const int *, const double *, const double *, const double *, double *,
                                          double *, const MgSteps<double> &, const DevState *,
                                          const MgTransfer<double> *, const double *, double *,
                                          const MgFirst<double> *);
template void launch_mg_smooth_tb<float>(hipStream_t, int, int, int, const Coef<float> &, const int8_t *, const int *,
                                         const float *, const float *, const float *, float *, float *,
                                         const MgSteps<float> &, const DevState *, const MgTransfer<float> *,
                                         const float *, float *, const MgFirst<float> *);
template void launch_mg_restrict<double>(hipStream_t, const MgTransfer<double> &, const double *, double *,
                                         const MgFirst<double> &);
template void launch_mg_restrict<float>(hipStream_t, const MgTransfer<float> &, const float *, float *,
                                        const MgFirst<float> &);
template void launch_mg_diag<double>(hipStream_t, int, int, int, const Coef<double> &, const int8_t *, const int *,
                                     const double *, double *);
template void launch_mg_diag<float>(hipStream_t, int, int, int, const Coef<float> &, const int8_t *, const int *,
                                    const float *, float *);
template void launch_mg_resid_restrict<double>(hipStream_t, const Geom &, const Tiling &, const Coef<double> &, const uint32_t *,
                                              const double *, const double *, const double *, const MgTransfer<double> &,
                                              double *, const MgFirst<double> &, const DevState *);
template void launch_mg_resid_restrict<float>(hipStream_t, const Geom &, const Tiling &, const Coef<float> &, const uint32_t *,
                                              const float *, const float *, const float *, const MgTransfer<float> &,
                                              float *, const MgFirst<float> &, const DevState *);
template void launch_mg_prolong_add<double>(hipStream_t, const MgTransfer<double> &, const uint32_t *, int,
                                            const double *, double *);
template void launch_mg_prolong_add<float>(hipStream_t, const MgTransfer<float> &, const uint32_t *, int, const float *,
                                           float *);

template MgMarches mg_marches<double>(const Geom &, const MgTransfer<double> &);
template MgMarches mg_marches<float>(const Geom &, const MgTransfer<float> &);
template bool mg_pair_pays<double>(const Geom &);
template bool mg_pair_pays<float>(const Geom &);
template bool mg_second_pays<double>(const Geom &);
template bool mg_second_pays<float>(const Geom &);
template void launch_mg_pair<double>(const Launch &, const Tiling &, const Coef<double> &, const Irr<double> &, const double *, const double *,
                                     double *, double *, double, double, double, const DevState *, const hipEvent_t *);
template void launch_mg_pair<float>(const Launch &, const Tiling &, const Coef<float> &, const Irr<float> &, const float *, const float *,
                                    float *, float *, double, double, double, const DevState *, const hipEvent_t *);

template void launch_mg_second<double>(const Launch &, const Tiling &, const Coef<double> &, const Irr<double> &, const double *,
                                       const double *, double *, double, double, double, const DevState *, const hipEvent_t *);
template void launch_mg_second<float>(const Launch &, const Tiling &, const Coef<float> &, const Irr<float> &, const float *,
                                      const float *, float *, double, double, double, const DevState *, const hipEvent_t *);

}  // namespace cps
