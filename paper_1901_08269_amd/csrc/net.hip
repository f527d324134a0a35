// net.hip -- the learned warm start: a 4-level 3D convolutional encoder-decoder on the
// 4x-coarsened grid, trained on solutions that the solver itself produces.
//
// Network (channels c0..c3, 3 input channels f, phi, g; one output): per level two 3x3x3
// convolutions with bias and ReLU; 2x2x2 average pooling between encoder levels; nearest
// x2 upsampling and concatenation [upsampled, skip] on the way up; a 1x1x1 head.
// Parameters (FP32 master copy, flat): per 3x3x3 layer W[co][ci][kz][ky][kx] then b[co],
// in the order E0a E0b E1a E1b E2a E2b E3a E3b D2a D2b D1a D1b D0a D0b; then the head's
// c0 weights and its bias.
//
// Device layout: activations are BF16, voxel-major [b][z][y][x][C] with C a multiple of 16
// (the 3 input channels are zero-padded to 16).  3x3x3 weights are BF16 [co][tap][ci].
// Convolutions are implicit GEMMs on the matrix cores: v_mfma_f32_16x16x16bf16 with FP32
// accumulation; a wavefront computes 16 voxels x (16 NG) output channels.  The data
// gradient is the same kernel with tap-flipped, channel-transposed weights; the weight
// gradient is an MFMA GEMM over voxels with LDS-staged tiles and a fixed-order reduction
// over voxel chunks.  Gradients entering each 3x3x3 layer are rounded to BF16 (the MFMA
// operand type); everything else in the backward pass is FP32.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "cps.h"
#include "cps_device.h"
#include "cps_host.h"

namespace cpsnet {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t bf16;

constexpr int NLAYER = 14;

// round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16 f2bf(float f) { return __builtin_bit_cast(bf16, static_cast<__bf16>(f)); }
__device__ __forceinline__ float bf2f(bf16 b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ bf16x4 load4(const bf16 *p)
{
    return *reinterpret_cast<const bf16x4 *>(p);
}

// ---------------------------------------------------------------------------------------
// 3x3x3 convolution (zero padding): Y[v][co] = act(bias[co] + sum_{tap,ci} W[co][tap][ci] X[v+tap][ci])
// ---------------------------------------------------------------------------------------
// Work items (run, part) in one grid of NXCD x per x parts blocks: the blocks of one XCD
// (consecutive ones go to the eight XCDs in turn) take a contiguous range of runs, all parts
// of a run one after another, so that the rows that neighbouring runs and the parts of one
// run share are read into that XCD's L2 once.
struct RunPart {
    int run, part;
};
inline unsigned run_blocks(size_t runs, int parts) { return (unsigned)((runs + cps::NXCD - 1) / cps::NXCD * cps::NXCD * parts); }
__device__ __forceinline__ RunPart run_of_block(int runs, int parts)
{
    const int per = (runs + cps::NXCD - 1) / cps::NXCD, k = (int)blockIdx.x / cps::NXCD;
    const int r = k / parts;
    return RunPart{((int)blockIdx.x % cps::NXCD) * per + r, k - r * parts};
}

// Rows of 16 channels staged in LDS for a run of voxels [v, v + len) and its tap neighbours of
// one z-offset: tap (dy, dx) of the run's l-th voxel is row l + dy * dys + dx.  One contiguous
// range of len + 2 n + 2 voxels holds all nine (dys = n); where 2 n + 2 rows more than the
// run's own would cost more than three ranges of len + 2, one per dy (dys = len + 2).
struct TapRows {
    int dys, seg, nseg;      // row stride of dy, rows of a range, ranges
};
inline TapRows tap_rows(int n, int len)
{
    if (2 * n + 2 + len <= 3 * (len + 2)) return TapRows{n, len + 2 * n + 2, 1};
    return TapRows{len + 2, len + 2, 3};
}
// rows of z-offset dz (0 .. 2) of the voxels from v on: 16 channels from channel c of X
// (voxel pitch C) as two 16-byte halves; rows outside the tensor are zero
__device__ __forceinline__ void stage_taps(const TapRows &tr, int n, int V, int v, int dz, int C, int c,
                                           const bf16 *__restrict__ X, uint4 *rows, int tid, int nt)
{
    for (int q = 0; q < tr.nseg; ++q) {
        const int u0 = v + (dz - 1) * n * n + (tr.nseg == 1 ? -n : (q - 1) * n) - 1;
        const bf16 *src = X + (ptrdiff_t)u0 * C + c;
        for (int h = tid; h < 2 * tr.seg; h += nt) {
            uint4 val{0u, 0u, 0u, 0u};
            if ((unsigned)(u0 + (h >> 1)) < (unsigned)V)
                val = *reinterpret_cast<const uint4 *>(src + (unsigned)((h >> 1) * C + 8 * (h & 1)));
            rows[2 * q * tr.seg + h] = val;
        }
    }
}

// What a convolution does with its sums:
//   CONV_ACT    Y (BF16) = ReLU(sum + bias)                                      (forward)
//   CONV_GATE   Y (BF16) = sum where the activation gate[v][co] > 0, else 0: the gradient
//               entering the layer that made this layer's input      (data gradient, odd layers)
//   CONV_F32    Y (FP32) = sum                            (data gradient of a pooled input)
//   CONV_SPLIT  channels below c_lo to Y (FP32, pitch c_lo), the others to Y2 (FP32): the two
//               parts of an upsampled and concatenated input
enum { CONV_ACT = 0, CONV_GATE = 1, CONV_F32 = 2, CONV_SPLIT = 3 };
struct ConvOut {
    const float *bias;
    const bf16 *gate;
    bf16 *yb;
    float *yf, *yf2;
    int c_lo;
};

// A block computes 64 M voxels x 16 NG output channels; wave w the 16 M voxels from 16 M w on.
// Sums run over (z-offset, channel slice, tap in the plane), a fixed order whatever NG and M:
// for each z-offset and 16-channel slice the block stages the rows of X that the nine taps of
// its voxels reach and the nine taps' weights, so a row is read from memory once per slice
// and a weight once per block; a wave's weight operands are read from LDS once for its M
// voxel groups.  Taps outside the grid are zeroed by the voxel's tap mask (one voxel per
// thread, exchanged through LDS: index divisions are what a block would otherwise spend most
// of its vector instructions on).  Per MFMA the kernel reads 1 / NG + 1 / M operands from LDS.
// In LDS the four 4-channel quarters of the rows lie in planes of their own (quarter q of row r
// at 8 (q pitch + r) bytes): the lanes of an operand read, 16 rows by four quarters, then cover
// whole runs of banks, where rows of 32 bytes had put eight rows on the same banks (70 % of the
// LDS cycles were conflicts).
// Measured at 64^3, batch 8, all 27 convolutions of a training step: 5.75 ms with the operands
// of every 16 voxels loaded from memory, 2.39 ms with staged 32-byte rows, 1.35 ms here.
__host__ __device__ __forceinline__ constexpr int quarter_pitch(int rows) { return ((rows + 15) & ~31) + 16; }   // 16 mod 32, >= rows
__device__ __forceinline__ void put_row_half(uint2 *p, int pitch, int h, uint4 v)
{
    uint2 *d = p + 2 * (h & 1) * pitch + (h >> 1);
    d[0] = uint2{v.x, v.y};
    d[pitch] = uint2{v.z, v.w};
}
template <int NG, int M, int OUT>
__global__ void __launch_bounds__(256) k_conv3(int n, int V, int Cin, int Cout, TapRows tr, const bf16 *__restrict__ X,
                                               const bf16 *__restrict__ Wk, ConvOut O)
{
    extern __shared__ uint4 lds[];
    __shared__ unsigned masks[64 * M];
    constexpr int WP = quarter_pitch(9 * 16 * NG);
    const int xp = quarter_pitch(tr.nseg * tr.seg);
    uint2 *xs = reinterpret_cast<uint2 *>(lds), *ws = xs + 4 * xp;     // ws: [9][16 NG] rows of 16 weights
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int row = lane & 15, kq = lane >> 4;
    const RunPart rp = run_of_block((V + 64 * M - 1) / (64 * M), Cout / 16 / NG);
    const int vb = rp.run * (64 * M), g0 = rp.part * NG;
    if (vb >= V) return;
    if (tid < 64 * M) {
        // bit t: tap t of voxel vb + tid lies in the grid
        const unsigned un = (unsigned)n, v = (unsigned)(vb + tid), vy = v / un, vz = vy / un;
        const unsigned x = v - vy * un, y = vy - vz * un, z = vz % un;
        const unsigned bx = (x > 0 ? 1u : 0u) | 2u | (x < un - 1 ? 4u : 0u);
        const unsigned by = (y > 0 ? bx : 0u) | bx << 3 | (y < un - 1 ? bx << 6 : 0u);
        masks[tid] = (z > 0 ? by : 0u) | by << 9 | (z < un - 1 ? by << 18 : 0u);
    }
    f32x4 acc[M][NG];
#pragma unroll
    for (int q = 0; q < M; ++q)
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[q][g] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint2 *xw = xs + kq * xp + 16 * M * wv + row, *ww = ws + kq * WP + row;
    // slice sl = (tz, c0).  With few voxels per block (M < 4: the coarse levels, whose launches
    // do not fill the GPU and wait out each slice's loads) its rows and weights are loaded into
    // registers while the slice before it is computed: 15 -> 9 us for M = 1.  With M = 4 the
    // registers cost more blocks in flight than that gains (119 -> 137 us).
    constexpr bool AHEAD = M < 4;
    constexpr int NX = AHEAD ? (6 * (64 * M + 2) + 255) / 256 : 1, NW = AHEAD ? (9 * 32 * NG + 255) / 256 : 1;
    const int nh = 2 * tr.nseg * tr.seg, nsl = 3 * (Cin / 16);
    // half h & 1 of row h >> 1 of the slice's rows of X, of its rows of weights
    auto x_half = [&](int tz, int c0, int h) {
        int u = vb + (tz - 1) * n * n - (tr.nseg == 1 ? n : 0) - 1 + (h >> 1);
        if (tr.nseg == 3) {                                    // ranges of one dy each
            const int q = (h >= 2 * tr.seg) + (h >= 4 * tr.seg);
            u += (q - 1) * n - q * tr.seg;
        }
        uint4 v{0u, 0u, 0u, 0u};
        if (h < nh && (unsigned)u < (unsigned)V)
            v = *reinterpret_cast<const uint4 *>(X + (size_t)(unsigned)u * Cin + c0 + 8 * (h & 1));
        return v;
    };
    auto w_half = [&](int tz, int c0, int h) {
        const int t9 = h / (32 * NG), co = (h >> 1) % (16 * NG);
        const bf16 *wsrc = Wk + ((size_t)16 * g0 * 27 + tz * 9) * Cin + c0;
        return *reinterpret_cast<const uint4 *>(wsrc + (unsigned)((co * 27 + t9) * Cin + 8 * (h & 1)));
    };
    uint4 xr[NX], wr[NW];
    auto fetch = [&](int tz, int c0) {
#pragma unroll
        for (int k = 0; k < NX; ++k) xr[k] = x_half(tz, c0, tid + 256 * k);
#pragma unroll
        for (int k = 0; k < NW; ++k) wr[k] = w_half(tz, c0, min(tid + 256 * k, 9 * 32 * NG - 1));
    };
    if (AHEAD) fetch(0, 0);
    int tz = 0, c0 = 0;
    for (int sl = 0; sl < nsl; ++sl) {
        if (AHEAD) {
#pragma unroll
            for (int k = 0; k < NX; ++k)
                if (tid + 256 * k < nh) put_row_half(xs, xp, tid + 256 * k, xr[k]);
#pragma unroll
            for (int k = 0; k < NW; ++k)
                if (tid + 256 * k < 9 * 32 * NG) put_row_half(ws, WP, tid + 256 * k, wr[k]);
        } else {
            for (int h = tid; h < nh; h += 256) put_row_half(xs, xp, h, x_half(tz, c0, h));
            for (int h = tid; h < 9 * 32 * NG; h += 256) put_row_half(ws, WP, h, w_half(tz, c0, h));
        }
        __syncthreads();
        const int tz_now = tz;
        c0 += 16;
        if (c0 == Cin) {
            c0 = 0;
            ++tz;
        }
        if (AHEAD && sl + 1 < nsl) fetch(tz, c0);
        {
            bf16x4 w[9][NG];
#pragma unroll
            for (int t9 = 0; t9 < 9; ++t9)
#pragma unroll
                for (int g = 0; g < NG; ++g) w[t9][g] = __builtin_bit_cast(bf16x4, ww[(t9 * NG + g) * 16]);
#pragma unroll
            for (int q = 0; q < M; ++q) {
                const int vm = (int)(masks[16 * (M * wv + q) + row] >> (9 * tz_now));
#pragma unroll
                for (int t9 = 0; t9 < 9; ++t9) {
                    uint2 a = xw[16 * q + (t9 / 3) * tr.dys + t9 % 3];
                    const unsigned k = (unsigned)((vm << (31 - t9)) >> 31);
                    a.x &= k;
                    a.y &= k;
#pragma unroll
                    for (int g = 0; g < NG; ++g)
                        acc[q][g] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a), w[t9][g],
                                                                              acc[q][g], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    // D[voxel 4 kq + i][co = row]
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int co = (g0 + g) * 16 + row;
        const float bco = OUT == CONV_ACT ? O.bias[co] : 0.f;
        // CONV_SPLIT: c_lo is a multiple of 16, so a group lies on one side
        const bool lo = OUT != CONV_SPLIT || co < O.c_lo;
        float *yf = lo ? O.yf : O.yf2;
        const int pitch = OUT != CONV_SPLIT ? Cout : (lo ? O.c_lo : Cout - O.c_lo), cc = lo ? co : co - O.c_lo;
#pragma unroll
        for (int q = 0; q < M; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int vo = vb + 16 * (M * wv + q) + 4 * kq + i;
                if (vo >= V) continue;
                const size_t e = (size_t)vo * pitch + cc;
                float val = acc[q][g][i] + bco;
                if (OUT == CONV_ACT) O.yb[e] = f2bf(val > 0.f ? val : 0.f);
                else if (OUT == CONV_GATE) O.yb[e] = bf2f(O.gate[e]) > 0.f ? f2bf(val) : (bf16)0;
                else yf[e] = val;
            }
    }
}

// ---------------------------------------------------------------------------------------
// weight gradient: P[chunk][co][tap][ci] = sum_{v in chunk} G[v][co] X[v+tap][ci]
// ---------------------------------------------------------------------------------------
// voxels per block: enough blocks to fill the GPU (about 2048 with the 27 taps), at most 4096
// voxels (fewer chunk partials to reduce), a multiple of 64
inline int wgrad_chunk(int V)
{
    const int c = (int)std::min<long>(4096, std::max<long>(256, (long)V * 27 / 2048));
    return (c + 63) / 64 * 64;
}
// db[c] = sum_v G[v][c] in two fixed-order passes.  Pass 1: COLSUM_PARTS parts; lane vl of a
// part adds every lanes-th voxel of the part's stride per channel (lanes = 256 / C), and the
// part's lanes are added per channel in lane order.  A thread takes eight channels of one lane
// (16-byte loads, eight of them in flight), a wavefront two parts.  The parts run in blocks of
// their own after the weight gradient's, in its launch, whose wavefronts leave the memory idle
// (us of a training step for the 14 layers in launches of their own: 137 at 64^3, batch 8, 42 at
// 16^3, batch 4).  Pass 2 (k_grad_final) adds the part sums.
constexpr int COLSUM_PARTS = 512;
constexpr int COLSUM_LDS = 256;          // floats per part of a block
__device__ __forceinline__ void colsum_part(int p, int V, int C, const bf16 *__restrict__ G, float *__restrict__ part,
                                            float *sh)
{
    const int lanes = 256 / C, c8 = C / 8;                 // C <= 64: at most 32 threads per part
    const int t = (int)threadIdx.x & 31, vl = t / c8, c = 8 * (t - vl * c8);
    if (vl < lanes && p < COLSUM_PARTS) {
        float s[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] = 0.f;
        const size_t step = (size_t)COLSUM_PARTS * lanes;
        auto add = [&](uint4 w) {
            const unsigned u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                s[2 * j] += __uint_as_float(u[j] << 16);
                s[2 * j + 1] += __uint_as_float(u[j] & 0xFFFF0000u);
            }
        };
        size_t v = (size_t)p * lanes + vl;
        for (; v + 7 * step < (size_t)V; v += 8 * step) {
            uint4 w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = *reinterpret_cast<const uint4 *>(G + (v + k * step) * C + c);
#pragma unroll
            for (int k = 0; k < 8; ++k) add(w[k]);
        }
        for (; v < (size_t)V; v += step) add(*reinterpret_cast<const uint4 *>(G + v * C + c));
#pragma unroll
        for (int j = 0; j < 8; ++j) sh[vl * C + c + j] = s[j];
    }
    __syncthreads();
    if (p >= COLSUM_PARTS) return;
    for (int q = t; q < C; q += 32) {
        float acc = 0.f;
        for (int l = 0; l < lanes; ++l) acc += sh[l * C + q];
        part[(size_t)p * C + q] = acc;
    }
}

constexpr int WG_VS = 256;       // voxels staged in LDS per round: sixteen 16-voxel MFMA steps
constexpr int WG_RED_TAPS = 3;   // taps per dz whose wave sums are exchanged at a time (SPLIT)

// Four consecutive rows (voxels) of one column (channel) from rows of 16 BF16 in LDS: lane
// (m, kq) of a wavefront receives column m of rows 4 kq .. 4 kq + 3 after row r0 -- the K-major
// operand of the voxel GEMM -- by the transposing LDS read, for which lane m of each group of
// 16 points at four columns of row m / 4.
__device__ __forceinline__ bf16x4 load_rows4(const bf16 *rows, int r0, int m, int kq)
{
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const bf16 *p = rows + (r0 + 4 * kq + (m >> 2)) * 16 + 4 * (m & 3);
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_bf16x4 *)p);
}

__device__ __forceinline__ bf16x4 mask4(bf16x4 a, uint2 k)
{
    uint2 u = __builtin_bit_cast(uint2, a);
    u.x &= k.x;
    u.y &= k.y;
    return __builtin_bit_cast(bf16x4, u);
}

// A block takes one chunk of voxels and, of the 16 x 16 output tiles (co, ci), either all
// those of one ci group (a wave per co group and dz) or, for layers with fewer
// than four tiles (SPLIT: the 16-channel layers on the largest grids), one tile,
// whose 16-voxel steps go round four waves per dz; the four sums are added in wave order.
// A wave holds the nine taps of its dz (36 accumulator registers).  WG_VS voxels of G and the
// rows of X that their 27 taps reach are staged at a time; both MFMA operands are K-major
// (voxels) and come from the transposing LDS read.  A tap outside the grid is dropped by
// zeroing G's voxels (masks per voxel and side of the grid, staged with them), so the staged
// rows serve every tap.  The kernel is bound by LDS reads: 15 (9 of X, 1 of G, 5 masks) for
// nine MFMAs.
// Measured at 64^3, batch 8: 734 us per layer on average for the version that staged X once
// per tap and gathered its operands by 2-byte LDS reads, 83 us for this one (10.3 -> 1.16 ms of a training step).
// SPLIT is held to the registers of six waves per SIMD (two blocks a CU), which spills 11 of them: 168 us
// a launch at 64^3, batch 8 against 205 without; the other form keeps its 91 (64 us with the limit, 56 without).
template <bool SPLIT>
__global__ void __launch_bounds__(768, SPLIT ? 6 : 1) k_wgrad(int n, int V, int Cin, int Cout, int wchunk, TapRows tr,
                                               const bf16 *__restrict__ G, const bf16 *__restrict__ X,
                                               float *__restrict__ P, int nblocks, float *__restrict__ bpart)
{
    extern __shared__ uint4 lds[];
    if ((int)blockIdx.x >= nblocks) {                          // the blocks after: the bias gradient's parts
        const int h = (int)threadIdx.x >> 5, p = ((int)blockIdx.x - nblocks) * ((int)blockDim.x >> 5) + h;
        colsum_part(p, V, Cout, G, bpart, reinterpret_cast<float *>(lds) + COLSUM_LDS * h);
        return;
    }
    const int tci = Cin / 16, tco = SPLIT ? 1 : Cout / 16;    // tco: co groups of the block
    const int zrows = tr.nseg * tr.seg;                        // rows of X per dz
    uint4 *xs = lds, *gs = lds + 2 * 3 * zrows;                // [3][zrows], [tco][WG_VS] rows
    uint16_t *mk = reinterpret_cast<uint16_t *>(gs + 2 * tco * WG_VS);   // [6][WG_VS]
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, kq = lane >> 4;
    const RunPart rp = run_of_block((V + wchunk - 1) / wchunk, SPLIT ? tci * (Cout / 16) : tci);
    const int chunk = rp.run, cig = SPLIT ? rp.part % tci : rp.part;
    const int cog0 = SPLIT ? rp.part / tci : 0;                // first co group of the block
    if (chunk * (long)wchunk >= V) return;
    const int wz = wv % 3, wq = wv / 3;                        // the wave's dz; co group or step residue
    const bf16 *xw = reinterpret_cast<const bf16 *>(xs + 2 * wz * zrows);
    const bf16 *gw = reinterpret_cast<const bf16 *>(gs + (SPLIT ? 0 : 2 * wq * WG_VS));
    f32x4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int vbeg = chunk * wchunk, vend = min(vbeg + wchunk, V);
    for (int vs = vbeg; vs < vend; vs += WG_VS) {
        for (int dz = 0; dz < 3; ++dz)
            stage_taps(tr, n, V, vs, dz, Cin, 16 * cig, X, xs + 2 * dz * zrows, tid, nt);
        for (int h = tid; h < 2 * tco * WG_VS; h += nt) {
            const int g = h / (2 * WG_VS), r = (h >> 1) % WG_VS, v = vs + r;
            uint4 val{0u, 0u, 0u, 0u};
            if (v < vend)
                val = *reinterpret_cast<const uint4 *>(G + (size_t)v * Cout + 16 * (cog0 + g) + 8 * (h & 1));
            gs[h] = val;
        }
        // x, y, z of the stage's voxels from those of its first one: the quotients are of numbers
        // below n + WG_VS, exact in FP32 with the half added
        const float inv = 1.f / (float)n;
        const int vx0 = vs % n, vy0 = (vs / n) % n, vz0 = (vs / (n * n)) % n;
        for (int r = tid; r < WG_VS; r += nt) {
            const int qx = (int)(((float)(vx0 + r) + 0.5f) * inv), x = vx0 + r - qx * n;
            const int qy = (int)(((float)(vy0 + qx) + 0.5f) * inv), y = vy0 + qx - qy * n;
            const int qz = (int)(((float)(vz0 + qy) + 0.5f) * inv), z = vz0 + qy - qz * n;
            mk[0 * WG_VS + r] = x > 0 ? 0xFFFFu : 0u;
            mk[1 * WG_VS + r] = x < n - 1 ? 0xFFFFu : 0u;
            mk[2 * WG_VS + r] = y > 0 ? 0xFFFFu : 0u;
            mk[3 * WG_VS + r] = y < n - 1 ? 0xFFFFu : 0u;
            mk[4 * WG_VS + r] = z > 0 ? 0xFFFFu : 0u;
            mk[5 * WG_VS + r] = z < n - 1 ? 0xFFFFu : 0u;
        }
        __syncthreads();
        const int nst = (min(WG_VS, vend - vs) + 15) / 16;
        for (int ks = SPLIT ? wq : 0; ks < nst; ks += SPLIT ? 4 : 1) {
            const int r0 = 16 * ks;
            auto side = [&](int q) { return *reinterpret_cast<const uint2 *>(mk + q * WG_VS + r0 + 4 * kq); };
            bf16x4 a = load_rows4(gw, r0, m, kq);                 // A[co][v]
            if (wz != 1) a = mask4(a, side(wz == 0 ? 4 : 5));
            const uint2 x0 = side(0), x2 = side(1);
            const bf16x4 ay[3] = {mask4(a, side(2)), a, mask4(a, side(3))};
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int dy = t / 3, dx = t % 3;
                const bf16x4 am = dx == 0 ? mask4(ay[dy], x0) : (dx == 2 ? mask4(ay[dy], x2) : ay[dy]);
                const bf16x4 b = load_rows4(xw, r0 + dy * tr.dys + dx, m, kq);   // B[v][ci]
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(am, b, acc[t], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    if (SPLIT) {
        f32x4 *red = reinterpret_cast<f32x4 *>(lds);            // [3 waves][3 dz][WG_RED_TAPS][64]
#pragma unroll
        for (int t0 = 0; t0 < 9; t0 += WG_RED_TAPS) {
            if (wq > 0)
#pragma unroll
                for (int t = 0; t < WG_RED_TAPS; ++t) red[(((wq - 1) * 3 + wz) * WG_RED_TAPS + t) * 64 + lane] = acc[t0 + t];
            __syncthreads();
            if (wq == 0)
#pragma unroll
                for (int t = 0; t < WG_RED_TAPS; ++t)
                    for (int w = 0; w < 3; ++w) acc[t0 + t] += red[((w * 3 + wz) * WG_RED_TAPS + t) * 64 + lane];
            __syncthreads();
        }
        if (wq > 0) return;
    }
    const int cog = SPLIT ? cog0 : wq;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int co = cog * 16 + 4 * kq + i, ci = cig * 16 + m;   // D[co][ci]
            P[(((size_t)chunk * Cout + co) * 27 + 9 * wz + t) * Cin + ci] = acc[t][i];
        }
}

// sum over chunks (fixed order) into the canonical gradient W[co][ci][tap] (ci < ci_real).
// The order is sequential per output and the outputs are few, so the loads of 32 chunks are
// issued before their additions (one memory round trip for 32 chunks instead of one for each).
__device__ __forceinline__ void wgrad_reduce(int block, int nchunk, int Cin, int Cout, int ci_real,
                                             const float *__restrict__ P, float *__restrict__ gW)
{
    constexpr int NB = 32;
    // thread order (co, tap, ci): consecutive threads read consecutive partials of a chunk
    int q = block * (int)blockDim.x + (int)threadIdx.x;
    int total = Cout * ci_real * 27;
    if (q >= total) return;
    int ci = q % ci_real, tap = (q / ci_real) % 27, co = q / (27 * ci_real);
    const float *p = P + ((size_t)co * 27 + tap) * Cin + ci;
    const size_t pitch = (size_t)Cout * 27 * Cin;
    float s = 0.f;
    int c = 0;
    for (; c + NB <= nchunk; c += NB) {
        float v[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) v[u] = p[(size_t)(c + u) * pitch];
#pragma unroll
        for (int u = 0; u < NB; ++u) s += v[u];
    }
    for (; c < nchunk; ++c) s += p[(size_t)c * pitch];
    gW[((size_t)co * ci_real + ci) * 27 + tap] = s;
}

// All layers' gradients from their partials in one launch: a layer's first wblocks blocks sum its
// weight gradient over chunks (wgrad_reduce), the C blocks after them one channel's bias gradient
// each (thread t adds parts t, t + 256, ...; then a tree in LDS).  Every layer's partials are kept
// until here: a launch per layer was bound by its own latency (us for the 14 layers: 16^3, batch 4
// 11 against 57; 64^3, batch 8 71 against 152).
struct GradLayer {
    int block0, wblocks, nchunk, cip, co, ci;   // block0: the layer's first block
    const float *P, *part;
    float *gW, *gb;
};
struct GradList {
    GradLayer l[NLAYER];
};
__global__ void __launch_bounds__(256) k_grad_final(GradList list)
{
    __shared__ float sh[256];
    int q = 0;
#pragma unroll
    for (int i = 1; i < NLAYER; ++i) q = (int)blockIdx.x >= list.l[i].block0 ? i : q;
    const GradLayer L = list.l[q];
    const int block = (int)blockIdx.x - L.block0;
    if (block < L.wblocks) {
        wgrad_reduce(block, L.nchunk, L.cip, L.co, L.ci, L.P, L.gW);
        return;
    }
    const float *__restrict__ part = L.part;
    float *__restrict__ gb = L.gb;
    const int c = block - L.wblocks, t = (int)threadIdx.x, Cout = L.co;
    float acc = 0.f;
    for (int b = t; b < COLSUM_PARTS; b += 256) acc += part[(size_t)b * Cout + c];
    sh[t] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o) sh[t] += sh[t + o];
        __syncthreads();
    }
    if (t == 0) gb[c] = sh[0];
}

// ---------------------------------------------------------------------------------------
// elementwise pieces
// ---------------------------------------------------------------------------------------
// the 16 channels of a voxel as two 16-byte accesses
__device__ __forceinline__ void load16(const bf16 *p, bf16 (&o)[16])
{
    const uint4 a = reinterpret_cast<const uint4 *>(p)[0], b = reinterpret_cast<const uint4 *>(p)[1];
    const unsigned w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        o[2 * j] = (bf16)(w[j] & 0xFFFFu);
        o[2 * j + 1] = (bf16)(w[j] >> 16);
    }
}
__device__ __forceinline__ void store16(bf16 *p, const bf16 (&o)[16])
{
    unsigned w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = (unsigned)o[2 * j] | (unsigned)o[2 * j + 1] << 16;
    reinterpret_cast<uint4 *>(p)[0] = uint4{w[0], w[1], w[2], w[3]};
    reinterpret_cast<uint4 *>(p)[1] = uint4{w[4], w[5], w[6], w[7]};
}

// g rounded to BF16 where the activation is positive (ReLU's gradient), 0 elsewhere
__device__ __forceinline__ bf16x4 gate4(float4 g, bf16x4 act)
{
    const float gv[4] = {g.x, g.y, g.z, g.w};
    bf16x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (short)(bf2f((bf16)act[j]) > 0.f ? f2bf(gv[j]) : (bf16)0);
    return o;
}

// input [B][cin][n^3] (FP32, channels first) -> [V][16] BF16, channels >= cin zero
// (one voxel per thread)
__global__ void k_pack_input(int V, int n3, int cin, const float *__restrict__ in, bf16 *__restrict__ out)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    const int b = v / n3, r = v - b * n3;
    bf16 o[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) o[c] = c < cin ? f2bf(in[((size_t)b * cin + c) * n3 + r]) : (bf16)0;
    store16(out + (size_t)v * 16, o);
}

// 2x2x2 average pooling, [V][C] at n -> [V/8][C] at n/2; eight channels per thread, its eight voxels'
// 16-byte loads at once (us per level on average, against a channel per thread and 2-byte loads: 64^3,
// batch 8 7.4 / 15.6, 32^3, batch 8 3.4 / 4.4)
__global__ void __launch_bounds__(256) k_pool(int B, int n, int C, const bf16 *__restrict__ in, bf16 *__restrict__ out)
{
    const int m = n / 2, c8 = C / 8;
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (size_t)B * m * m * m * c8) return;
    const size_t vq = q / c8;
    const unsigned c = 8 * (unsigned)(q - vq * c8), v = (unsigned)vq, um = (unsigned)m;
    const unsigned vy = v / um, vz = vy / um, b = vz / um, x = v - vy * um, y = vy - vz * um, z = vz - b * um;
    union Eight {
        uint4 w;
        bf16 h[8];
    } ch[8], o8;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        const unsigned zz = 2 * z + (o >> 2), yy = 2 * y + ((o >> 1) & 1), xx = 2 * x + (o & 1);
        ch[o].w = *reinterpret_cast<const uint4 *>(in + ((((size_t)b * n + zz) * n + yy) * n + xx) * C + c);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float s = 0.f;
#pragma unroll
        for (int o = 0; o < 8; ++o) s += bf2f(ch[o].h[j]);
        o8.h[j] = f2bf(s * 0.125f);
    }
    *reinterpret_cast<uint4 *>(out + vq * C + c) = o8.w;
}

// gradient entering the 3x3x3 layer before a pooling (its output act at n, [V][C]): the skip
// connection's part gskip plus an eighth of the pooled cell's gradient, masked by the ReLU,
// rounded to BF16.  Four channels per thread.
__global__ void k_pool_bwd(int B, int n, int C, const float *__restrict__ gpool, const float *__restrict__ gskip,
                           const bf16 *__restrict__ act, bf16 *__restrict__ out)
{
    const int m = n / 2, c4 = C / 4;
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (size_t)B * n * n * n * c4) return;
    const size_t vq = q / c4;
    const unsigned c = 4 * (unsigned)(q - vq * c4), v = (unsigned)vq, un = (unsigned)n;
    const unsigned vy = v / un, vz = vy / un, b = vz / un, x = v - vy * un, y = vy - vz * un, z = vz - b * un;
    const float4 gp =
        *reinterpret_cast<const float4 *>(gpool + ((((size_t)b * m + z / 2) * m + y / 2) * m + x / 2) * C + c);
    const float4 gs = *reinterpret_cast<const float4 *>(gskip + vq * C + c);
    *reinterpret_cast<bf16x4 *>(out + vq * C + c) =
        gate4(float4{gs.x + gp.x * 0.125f, gs.y + gp.y * 0.125f, gs.z + gp.z * 0.125f, gs.w + gp.w * 0.125f},
              load4(act + vq * C + c));
}

// [up(lo) (C0), skip (C1)] at n = 2m; eight channels per thread
__global__ void k_upcat(int B, int m, int C0, int C1, const bf16 *__restrict__ lo, const bf16 *__restrict__ skip,
                        bf16 *__restrict__ out)
{
    const int n = 2 * m, C = C0 + C1, c8 = C / 8;
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (size_t)B * n * n * n * c8) return;
    const size_t vq = q / c8;
    const unsigned c = 8 * (unsigned)(q - vq * c8), v = (unsigned)vq, un = (unsigned)n;
    const bf16 *src;
    if (c >= (unsigned)C0) {
        src = skip + vq * C1 + (c - C0);
    } else {
        const unsigned vy = v / un, vz = vy / un, b = vz / un, x = v - vy * un, y = vy - vz * un, z = vz - b * un;
        src = lo + ((((size_t)b * m + z / 2) * m + y / 2) * m + x / 2) * C0 + c;
    }
    *reinterpret_cast<uint4 *>(out + vq * C + c) = *reinterpret_cast<const uint4 *>(src);
}

// gradient entering the 3x3x3 layer whose output act (at m, [u][C]) was upsampled: the sum of
// its eight children's gradients g (at n = 2m), masked by the ReLU, rounded to BF16.  Four
// channels per thread.
__global__ void k_up_bwd(int B, int m, int C, const float *__restrict__ g, const bf16 *__restrict__ act,
                         bf16 *__restrict__ out)
{
    const int n = 2 * m, c4 = C / 4;
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (size_t)B * m * m * m * c4) return;
    const size_t uq = q / c4;
    const unsigned c = 4 * (unsigned)(q - uq * c4), u = (unsigned)uq, um = (unsigned)m;
    const unsigned uy = u / um, uz = uy / um, b = uz / um, x = u - uy * um, y = uy - uz * um, z = uz - b * um;
    float4 ch[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        const unsigned zz = 2 * z + (o >> 2), yy = 2 * y + ((o >> 1) & 1), xx = 2 * x + (o & 1);
        ch[o] = *reinterpret_cast<const float4 *>(g + ((((size_t)b * n + zz) * n + yy) * n + xx) * C + c);
    }
    float4 s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        s.x += ch[o].x;
        s.y += ch[o].y;
        s.z += ch[o].z;
        s.w += ch[o].w;
    }
    *reinterpret_cast<bf16x4 *>(out + uq * C + c) = gate4(s, load4(act + uq * C + c));
}

// head: p[v] = hb + sum_c hw[c] act[v][c], HEAD_C channels
constexpr int HEAD_C = 16;
__global__ void k_head(int V, const bf16 *__restrict__ act, const float *__restrict__ hw, float *__restrict__ p)
{
    int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    bf16 a[HEAD_C];
    load16(act + (size_t)v * HEAD_C, a);
    float s = hw[HEAD_C];
#pragma unroll
    for (int c = 0; c < HEAD_C; ++c) s += hw[c] * bf2f(a[c]);
    p[v] = s;
}

// masked squared error: per-block partial sums of m (p - t)^2 and m
__global__ void k_loss_partial(int V, const float *__restrict__ p, const float *__restrict__ t,
                               const float *__restrict__ mask, double *__restrict__ part)
{
    __shared__ double s0[256], s1[256];
    double a = 0.0, w = 0.0;
    for (int v = blockIdx.x * 256 + threadIdx.x; v < V; v += gridDim.x * 256) {
        double m = mask ? (double)mask[v] : 1.0;
        double d = (double)p[v] - (double)t[v];
        a += m * d * d;
        w += m;
    }
    s0[threadIdx.x] = a;
    s1[threadIdx.x] = w;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            s0[threadIdx.x] += s0[threadIdx.x + o];
            s1[threadIdx.x] += s1[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = s0[0];
        part[2 * blockIdx.x + 1] = s1[0];
    }
}

constexpr int LOSS_BLOCKS = 256;
__global__ void __launch_bounds__(LOSS_BLOCKS) k_loss_final(const double *__restrict__ part, double *__restrict__ out)
{
    __shared__ double s0[LOSS_BLOCKS], s1[LOSS_BLOCKS];
    const int t = (int)threadIdx.x;
    s0[t] = part[2 * t];
    s1[t] = part[2 * t + 1];
    __syncthreads();
    for (int o = LOSS_BLOCKS / 2; o > 0; o >>= 1) {
        if (t < o) {
            s0[t] += s0[t + o];
            s1[t] += s1[t + o];
        }
        __syncthreads();
    }
    if (t == 0) {
        out[0] = s0[0] / s1[0];
        out[1] = s1[0];
    }
}

// head backward: dp = 2 m (p - t) / sum m; the gradient entering the last 3x3x3 layer, dp hw[c]
// masked by its ReLU and rounded to BF16; partials of dhw, dhb
constexpr int HEAD_BLOCKS = 512;    // blocks of the head's backward reduction
__global__ void __launch_bounds__(256) k_head_bwd(int V, const float *__restrict__ p, const float *__restrict__ t,
                                                  const float *__restrict__ mask, const double *__restrict__ lossw,
                                                  const bf16 *__restrict__ act, const float *__restrict__ hw,
                                                  bf16 *__restrict__ gb, float *__restrict__ part /*[gridDim][17]*/)
{
    constexpr int C = HEAD_C;
    __shared__ float sh[256][C + 1];
    const double inv = 1.0 / lossw[1];
    float loc[C + 1];
#pragma unroll
    for (int c = 0; c <= C; ++c) loc[c] = 0.f;
    for (int v = blockIdx.x * 256 + threadIdx.x; v < V; v += gridDim.x * 256) {
        float m = mask ? mask[v] : 1.f;
        float dp = (float)(2.0 * m * ((double)p[v] - (double)t[v]) * inv);
        bf16 a[C], o[C];
        load16(act + (size_t)v * C, a);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float av = bf2f(a[c]);
            o[c] = av > 0.f ? f2bf(dp * hw[c]) : (bf16)0;
            loc[c] += dp * av;
        }
        store16(gb + (size_t)v * C, o);
        loc[C] += dp;
    }
#pragma unroll
    for (int c = 0; c <= C; ++c) sh[threadIdx.x][c] = loc[c];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
            for (int c = 0; c <= C; ++c) sh[threadIdx.x][c] += sh[threadIdx.x + o][c];
        __syncthreads();
    }
    if (threadIdx.x <= C) part[(size_t)blockIdx.x * (C + 1) + threadIdx.x] = sh[0][threadIdx.x];
}

// one block per output (C weights and the bias): partials t, t + 256, ... then a tree
__global__ void __launch_bounds__(256) k_head_bwd_final(int nb, int C, const float *__restrict__ part,
                                                        float *__restrict__ g)
{
    __shared__ float sh[256];
    const int c = (int)blockIdx.x, t = (int)threadIdx.x;
    float s = 0.f;
    for (int b = t; b < nb; b += 256) s += part[(size_t)b * (C + 1) + c];
    sh[t] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o) sh[t] += sh[t + o];
        __syncthreads();
    }
    if (t == 0) g[c] = sh[0];
}

// Adam on the FP32 master parameters (Kingma & Ba), step t >= 1
__global__ void k_adam(size_t n, float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m1,
                       float *__restrict__ m2, float lr, float b1, float b2, float eps, float c1, float c2)
{
    size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    float gq = g[q];
    float a = b1 * m1[q] + (1.f - b1) * gq;
    float b = b2 * m2[q] + (1.f - b2) * gq * gq;
    m1[q] = a;
    m2[q] = b;
    w[q] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

// pack canonical W[co][ci][tap] (FP32) into BF16 Wk[co][tap][cip] and flipped Wf[ci][tap'][co],
// all layers in one launch (blockIdx.y: the layer)
struct PackLayer {
    int ci, co, cip;
    const float *W;
    bf16 *Wk, *Wf;
};
struct PackList {
    PackLayer l[NLAYER];
};
__global__ void k_pack_weights(PackList list)
{
    const PackLayer &L = list.l[blockIdx.y];
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= L.co * 27 * L.cip) return;
    int c = q % L.cip, tap = (q / L.cip) % 27, o = q / (27 * L.cip);
    float v = c < L.ci ? L.W[((size_t)o * L.ci + c) * 27 + tap] : 0.f;
    bf16 b = f2bf(v);
    L.Wk[q] = b;
    if (L.Wf && c < L.ci) L.Wf[((size_t)c * 27 + (26 - tap)) * L.co + o] = b;
}

// ---------------------------------------------------------------------------------------
// fine grid <-> coarse grid
// ---------------------------------------------------------------------------------------
// sums of g^2 and (f / 3 pi^2)^2 over all nodes (per-block partials; 1024 threads per
// block, 16-byte loads: a pass over two fine-grid FP64 arrays)
__global__ void __launch_bounds__(1024) k_scale_partial(size_t nn, const double *__restrict__ f,
                                                        const double *__restrict__ g, double *__restrict__ part)
{
    __shared__ double sh[1024];
    const double k = 1.0 / (3.0 * M_PI * M_PI);
    double s = 0.0;
    const size_t n2 = nn / 2;
    const double2 *f2 = reinterpret_cast<const double2 *>(f), *g2 = reinterpret_cast<const double2 *>(g);
    for (size_t e = (size_t)blockIdx.x * 1024 + threadIdx.x; e < n2; e += (size_t)gridDim.x * 1024) {
        const double2 a = g2[e], b = f2[e];
        const double b0 = b.x * k, b1 = b.y * k;
        s += (a.x * a.x + b0 * b0) + (a.y * a.y + b1 * b1);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && (nn & 1)) {
        const double a = g[nn - 1], b = f[nn - 1] * k;
        s += a * a + b * b;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_scale_final(int nb, size_t nn, const double *__restrict__ part, double *__restrict__ sigma)
{
    if (threadIdx.x || blockIdx.x) return;
    double s = 0.0;
    for (int b = 0; b < nb; ++b) s += part[b];
    double v = sqrt(s / (double)nn);
    sigma[0] = v > 0.0 ? v : 1.0;
}

// coarse cell (cx, cy, cz) <- means over fine interior nodes 1+4c .. 4+4c per direction:
// channel 0 f / (3 pi^2 sigma), 1 clamp(phi * nc / 8, -1, 1), 2 g / sigma; FP32 [1][3][nc^3]
__global__ void k_restrict(int nx, int ny, int nc, const double *__restrict__ f, const double *__restrict__ phi,
                           const double *__restrict__ g, const double *__restrict__ sigma, float *__restrict__ out)
{
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    int nc3 = nc * nc * nc;
    if (q >= nc3) return;
    int cx = q % nc, cy = (q / nc) % nc, cz = q / (nc * nc);
    double sf = 0.0, sp = 0.0, sg = 0.0;
    for (int dz = 0; dz < 4; ++dz)
        for (int dy = 0; dy < 4; ++dy)
            for (int dx = 0; dx < 4; ++dx) {
                size_t e = (size_t)(1 + 4 * cx + dx) + (size_t)nx * ((1 + 4 * cy + dy) + (size_t)ny * (1 + 4 * cz + dz));
                sf += f[e];
                sp += phi[e];
                sg += g[e];
            }
    const double inv = 1.0 / 64.0, s = sigma[0];
    out[q] = (float)(sf * inv / (3.0 * M_PI * M_PI * s));
    double ph = sp * inv * nc / 8.0;
    out[nc3 + q] = (float)(ph < -1.0 ? -1.0 : (ph > 1.0 ? 1.0 : ph));
    out[2 * nc3 + q] = (float)(sg * inv / s);
}

// target restriction: cell means over the same blocks of the solution's smooth extension
// (u at fluid nodes, g at nodes inside a body, phi <= 0), divided by sigma (FP32 [nc^3]).
// The solution itself is 0 inside the bodies; a cell mean that mixes those zeros with the
// fluid values interpolates badly next to the interface, where g continues u.
__global__ void k_restrict_u(int nx, int ny, int nc, const double *__restrict__ u, const double *__restrict__ phi,
                             const double *__restrict__ g, const double *__restrict__ sigma, float *__restrict__ out)
{
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nc * nc * nc) return;
    int cx = q % nc, cy = (q / nc) % nc, cz = q / (nc * nc);
    double s = 0.0;
    for (int dz = 0; dz < 4; ++dz)
        for (int dy = 0; dy < 4; ++dy)
            for (int dx = 0; dx < 4; ++dx) {
                const size_t e =
                    (size_t)(1 + 4 * cx + dx) + (size_t)nx * ((1 + 4 * cy + dy) + (size_t)ny * (1 + 4 * cz + dz));
                s += phi[e] > 0.0 ? u[e] : g[e];
            }
    out[q] = (float)(s / 64.0 / sigma[0]);
}

// u0 at fine nodes: trilinear interpolation in index space of the coarse cell values
// (cell c centred at fine index 2.5 + 4c), constant beyond the outer cell centres
// one thread per node: x from the thread index, y and z from the grid (no index divisions)
__global__ void k_prolong(int nx, int ny, int nz, int nc, const float *__restrict__ p, const double *__restrict__ sigma,
                          double *__restrict__ u0)
{
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x), j = (int)blockIdx.y, k = (int)blockIdx.z;
    if (i >= nx) return;
    const size_t e = (size_t)i + (size_t)nx * ((size_t)j + (size_t)ny * k);
    int idx[3] = {i, j, k};
    int c0[3];
    float w[3];
    for (int d = 0; d < 3; ++d) {
        float s = ((float)idx[d] - 2.5f) * 0.25f;
        s = fminf(fmaxf(s, 0.f), (float)(nc - 1));
        int c = (int)floorf(s);
        if (c > nc - 2) c = nc - 2;
        if (c < 0) c = 0;
        c0[d] = c;
        w[d] = s - (float)c;
    }
    double acc = 0.0;
    for (int o = 0; o < 8; ++o) {
        int ox = o & 1, oy = (o >> 1) & 1, oz = o >> 2;
        double ww = (ox ? w[0] : 1.f - w[0]) * (oy ? w[1] : 1.f - w[1]) * (oz ? w[2] : 1.f - w[2]);
        acc += ww * p[((c0[2] + oz) * nc + (c0[1] + oy)) * nc + (c0[0] + ox)];
    }
    u0[e] = acc * sigma[0];
}

}  // namespace cpsnet

// The sigma reduction of the restriction runs on SCALE_BLOCKS blocks whatever the grid size
// (grid-stride loop), so its scratch has a fixed size.
constexpr int SCALE_BLOCKS = 256;

// Scratch of cps_model_restrict_noalloc: [0, SCALE_BLOCKS) per-block partial sums of the
// sigma reduction, [SCALE_BLOCKS] sigma.  Every element is written before it is read in a
// call, so nothing needs clearing.  Each device holds one copy until the process ends; host
// code reaches it only through the address hipGetSymbolAddress returns for that device.
static __device__ __align__(256) double scratch[SCALE_BLOCKS + 1];

// =========================================================================================
// model object and its C-ABI
// =========================================================================================
using namespace cpsnet;

// solver internals needed by the restriction (defined in solver.hip)
extern "C++" int cps_internal_fields(cps_solver *s, const double **phi, const double **g, const double **f, int *nx,
                                     int *ny, int *nz, void **stream);

struct LayerInfo {
    int ci, co, cip, lvl;
    long off;    // offset of W in the flat parameters (bias follows)
    size_t part; // offset of the weight gradient's chunk partials
};

struct cps_model {
    cps_model_spec spec;
    hipStream_t stream = nullptr;
    LayerInfo L[NLAYER];
    long nparam = 0, head_off = 0;
    float *w = nullptr, *g = nullptr, *m1 = nullptr, *m2 = nullptr;   // flat FP32
    bf16 *Wk[NLAYER] = {}, *Wf[NLAYER] = {};
    bf16 *in[NLAYER] = {}, *out[NLAYER] = {};
    bool in_owned[NLAYER] = {};
    float *gskip[NLAYER] = {};  // gradient through the skip connections (layers 1, 3, 5), FP32
    float *gtmp = nullptr;      // data gradient of a pooled or upsampled input, FP32
    bf16 *gb = nullptr, *gb2 = nullptr;   // gradients entering two consecutive layers (BF16, masked)
    float *wpart = nullptr;    // weight-gradient chunk partials, layer by layer
    size_t wpart_n = 0;
    float *pred = nullptr, *inp = nullptr;
    float *arg[3] = {};         // copies of a call's inputs, targets and masks that are not in this device's memory
    double *lpart = nullptr, *lossv = nullptr, *sig = nullptr;
    float *hpart = nullptr;
    float *cpart = nullptr;    // bias-gradient column-sum partials (COLSUM_PARTS x 64 per layer)
    int adam_t = 0;
    int device = 0;             // the device current at creation (its stream's device)
    std::vector<void *> allocs;
};

namespace {

struct NetFail {
    int code;
};

void nck(hipError_t e)
{
    if (e != hipSuccess) throw NetFail{CPS_EDEVICE};
}

// an error that an earlier call of the program left behind (and reported then) is not this call's
void forget_errors() { (void)hipGetLastError(); }

inline unsigned nblk(size_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// Device address of `scratch` on device `dev`, looked up once per device with that device
// current (the previous current device is restored).
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
double *scratch_dev[MAX_DEVICES] = {};

double *scratch_address(int dev)
{
    if (dev < 0 || dev >= MAX_DEVICES) throw NetFail{CPS_EDEVICE};
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_dev[dev]) {
        int cur = 0;
        nck(hipGetDevice(&cur));
        if (cur != dev) nck(hipSetDevice(dev));
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != dev) nck(hipSetDevice(cur));
        if (e != hipSuccess || !p) throw NetFail{CPS_EDEVICE};
        scratch_dev[dev] = static_cast<double *>(p);
    }
    return scratch_dev[dev];
}

// The network input of the solver's problem (and the target's cell means of u), with the
// sigma reduction's partial sums in part[SCALE_BLOCKS] and sigma in sig[0] (device).
// The network's inputs for the fields phi, g, f of an nx x ny x nz grid, queued on the
// model's stream; with `wait` the call returns once they are complete.
int restrict_fields(cps_model *m, int nx, int ny, int nz, const double *phi, const double *g, const double *f,
                    const double *u, float *inputs, float *target, double *sigma, double *part, double *sig, bool wait)
{
    const int nc = m->spec.nc;
    if (nx - 2 != 4 * nc || ny - 2 != 4 * nc || nz - 2 != 4 * nc || m->spec.in_ch != 3) return CPS_EINVAL;
    const size_t nn = (size_t)nx * ny * nz;
    k_scale_partial<<<SCALE_BLOCKS, 1024, 0, m->stream>>>(nn, f, g, part);
    k_scale_final<<<1, 64, 0, m->stream>>>(SCALE_BLOCKS, nn, part, sig);
    k_restrict<<<nblk((size_t)nc * nc * nc), 256, 0, m->stream>>>(nx, ny, nc, f, phi, g, sig, inputs);
    if (u && target)
        k_restrict_u<<<nblk((size_t)nc * nc * nc), 256, 0, m->stream>>>(nx, ny, nc, u, phi, g, sig, target);
    nck(hipGetLastError());
    if (sigma) nck(hipMemcpyAsync(sigma, sig, sizeof(double), hipMemcpyDeviceToHost, m->stream));
    if (wait) nck(hipStreamSynchronize(m->stream));
    return CPS_OK;
}

int restrict_into(cps_model *m, cps_solver *s, const double *u, float *inputs, float *target, double *sigma,
                  double *part, double *sig)
{
    const double *phi, *g, *f;
    int nx, ny, nz;
    void *sst;
    cps_internal_fields(s, &phi, &g, &f, &nx, &ny, &nz, &sst);
    return restrict_fields(m, nx, ny, nz, phi, g, f, u, inputs, target, sigma, part, sig, true);
}

template <typename T>
T *nalloc(cps_model *m, size_t n)
{
    void *p = nullptr;
    if (hipMalloc(&p, (n ? n : 1) * sizeof(T)) != hipSuccess) throw NetFail{CPS_ENOMEM};
    m->allocs.push_back(p);
    nck(hipMemsetAsync(p, 0, (n ? n : 1) * sizeof(T), m->stream));
    return (T *)p;
}

// an array of n values that a call reads: in place, or copied into the model's buffer q (of `most`
// values, made on first use) where the kernels cannot read it
const float *readable(cps_model *m, const float *p, size_t n, int q, size_t most)
{
    if (!p || cps::device_array(p, n * sizeof(float), m->device)) return p;
    if (!m->arg[q]) m->arg[q] = nalloc<float>(m, most);
    nck(hipMemcpyAsync(m->arg[q], p, n * sizeof(float), hipMemcpyDefault, m->stream));
    return m->arg[q];
}

void layer_table(const int ch[4], int cin, LayerInfo L[NLAYER])
{
    const int lv[NLAYER] = {0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 1, 1, 0, 0};
    const int ci[NLAYER] = {cin, ch[0], ch[0], ch[1], ch[1], ch[2], ch[2], ch[3], ch[3] + ch[2], ch[2],
                            ch[2] + ch[1], ch[1], ch[1] + ch[0], ch[0]};
    const int co[NLAYER] = {ch[0], ch[0], ch[1], ch[1], ch[2], ch[2], ch[3], ch[3], ch[2], ch[2], ch[1], ch[1], ch[0], ch[0]};
    long off = 0;
    for (int q = 0; q < NLAYER; ++q) {
        L[q].ci = ci[q];
        L[q].co = co[q];
        L[q].cip = (ci[q] + 15) / 16 * 16;
        L[q].lvl = lv[q];
        L[q].off = off;
        off += (long)co[q] * ci[q] * 27 + co[q];
    }
}


int skip_of(int q) { return q == 8 ? 5 : (q == 10 ? 3 : 1); }

template <int NG, int M, int OUT>
void launch_conv_as(cps_model *m, int n, int V, int Cin, int Cout, const bf16 *X, const bf16 *W, const ConvOut &O)
{
    const TapRows tr = tap_rows(n, 64 * M);
    const size_t lds = 32 * ((size_t)quarter_pitch(tr.nseg * tr.seg) + quarter_pitch(9 * 16 * NG));
    const unsigned grid = run_blocks(nblk((size_t)V, 64 * M), Cout / 16 / NG);
    k_conv3<NG, M, OUT><<<grid, 256, lds, m->stream>>>(n, V, Cin, Cout, tr, X, W, O);
}

// Shape of the convolution's blocks: the widest of the listed ones (fewest LDS reads per
// MFMA first) whose launch still has CONV_MIN_BLOCKS blocks; the narrowest otherwise.
constexpr int CONV_MIN_BLOCKS = 512;
template <int OUT>
void launch_conv(cps_model *m, int n, int V, int Cin, int Cout, const bf16 *X, const bf16 *W, const ConvOut &O)
{
    const int groups = Cout / 16;
    auto fits = [&](int NG, int M) {
        return groups % NG == 0 && (size_t)nblk((size_t)V, 64 * M) * (groups / NG) >= (size_t)CONV_MIN_BLOCKS;
    };
#define CONV(NG, M) launch_conv_as<NG, M, OUT>(m, n, V, Cin, Cout, X, W, O)
    if (fits(3, 4)) CONV(3, 4);
    else if (fits(2, 4)) CONV(2, 4);
    else if (fits(3, 2)) CONV(3, 2);
    else if (fits(2, 2)) CONV(2, 2);
    else if (fits(1, 4)) CONV(1, 4);
    else if (fits(2, 1)) CONV(2, 1);
    else if (fits(1, 2)) CONV(1, 2);
    else CONV(1, 1);
#undef CONV
}

void launch_wgrad(cps_model *m, int n, int V, int Cin, int Cout, int wchunk, int nchunk, const bf16 *G, const bf16 *X,
                  float *part, float *bpart)
{
    const int tco = Cout / 16, tci = Cin / 16;
    const bool split = tco * tci < 4;
    const TapRows tr = tap_rows(n, WG_VS);
    const size_t rows = 3 * (size_t)tr.nseg * tr.seg + (split ? 1 : tco) * WG_VS;
    const size_t red = split ? sizeof(f32x4) * 9 * WG_RED_TAPS * 64 : 0;
    const int nt = split ? 768 : 192 * tco, groups = nt / 32;
    const size_t lds = std::max(std::max(rows * 32 + 6 * WG_VS * sizeof(uint16_t), red),
                                groups * COLSUM_LDS * sizeof(float));
    const void *fn = split ? reinterpret_cast<const void *>(&k_wgrad<true>) : reinterpret_cast<const void *>(&k_wgrad<false>);
    // more than 64 KB of LDS has to be asked for: from 26 / 69 / 112 / 154 cells per axis of the level on
    // with 64 / 48 / 32 / 16 output channels of the block (192 bytes per cell of a row, 8 KB per 16 channels)
    if (lds > 65536) nck(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int nblocks = (int)run_blocks(nchunk, split ? tco * tci : tci), grid = nblocks + (COLSUM_PARTS + groups - 1) / groups;
    if (split)
        k_wgrad<true><<<grid, nt, lds, m->stream>>>(n, V, Cin, Cout, wchunk, tr, G, X, part, nblocks, bpart);
    else
        k_wgrad<false><<<grid, nt, lds, m->stream>>>(n, V, Cin, Cout, wchunk, tr, G, X, part, nblocks, bpart);
}

void repack(cps_model *m)
{
    PackList list;
    size_t most = 0;
    for (int q = 0; q < NLAYER; ++q) {
        const LayerInfo &l = m->L[q];
        list.l[q] = PackLayer{l.ci, l.co, l.cip, m->w + l.off, m->Wk[q], q > 0 ? m->Wf[q] : nullptr};
        most = std::max(most, (size_t)l.co * 27 * l.cip);
    }
    k_pack_weights<<<dim3(nblk(most), NLAYER), 256, 0, m->stream>>>(list);
}

// pred = network(inp); inp, pred: device arrays of the caller's or the model's own
void forward(cps_model *m, int B, const float *inp, float *pred)
{
    const int nc = m->spec.nc;
    const int cin = m->spec.in_ch;
    int V0 = B * nc * nc * nc;
    k_pack_input<<<nblk((size_t)V0), 256, 0, m->stream>>>(V0, nc * nc * nc, cin, inp, m->in[0]);
    for (int q = 0; q < NLAYER; ++q) {
        const LayerInfo &l = m->L[q];
        const int n = nc >> l.lvl;
        const int V = B * n * n * n;
        if (q == 2 || q == 4 || q == 6) {
            k_pool<<<nblk((size_t)V * l.cip / 8), 256, 0, m->stream>>>(B, 2 * n, l.cip, m->out[q - 1], m->in[q]);
        } else if (q == 8 || q == 10 || q == 12) {
            int sk = skip_of(q);
            k_upcat<<<nblk((size_t)V * l.cip / 8), 256, 0, m->stream>>>(B, n / 2, m->L[q - 1].co, m->L[sk].co,
                                                                        m->out[q - 1], m->out[sk], m->in[q]);
        }
        ConvOut O{};
        O.bias = m->w + l.off + (long)l.co * l.ci * 27;
        O.yb = m->out[q];
        launch_conv<CONV_ACT>(m, n, V, l.cip, l.co, m->in[q], m->Wk[q], O);
    }
    k_head<<<nblk(V0), 256, 0, m->stream>>>(V0, m->out[NLAYER - 1], m->w + m->head_off, pred);
}

// after forward(m, B, ., m->pred)
void backward(cps_model *m, int B, const float *tgt, const float *msk)
{
    const int nc = m->spec.nc;
    const int V0 = B * nc * nc * nc;
    // loss
    k_loss_partial<<<LOSS_BLOCKS, 256, 0, m->stream>>>(V0, m->pred, tgt, msk, m->lpart);
    k_loss_final<<<1, LOSS_BLOCKS, 0, m->stream>>>(m->lpart, m->lossv);
    const int nhb = HEAD_BLOCKS;
    k_head_bwd<<<nhb, 256, 0, m->stream>>>(V0, m->pred, tgt, msk, m->lossv, m->out[NLAYER - 1], m->w + m->head_off,
                                           m->gb, m->hpart);
    k_head_bwd_final<<<HEAD_C + 1, 256, 0, m->stream>>>(nhb, HEAD_C, m->hpart, m->g + m->head_off);
    // gb: the gradient entering layer q (BF16, masked by its ReLU), made by the layer after it
    bf16 *gb = m->gb, *gnext = m->gb2;
    GradList grads{};
    for (int q = NLAYER - 1; q >= 0; --q, std::swap(gb, gnext)) {
        const LayerInfo &l = m->L[q];
        const int n = nc >> l.lvl;
        const int V = B * n * n * n;
        // weight and bias gradients
        const int wchunk = wgrad_chunk(V), nchunk = (V + wchunk - 1) / wchunk;
        float *wpart = m->wpart + l.part, *cpart = m->cpart + (size_t)q * COLSUM_PARTS * 64;
        launch_wgrad(m, n, V, l.cip, l.co, wchunk, nchunk, gb, m->in[q], wpart, cpart);
        grads.l[q] = GradLayer{0, (int)nblk((size_t)l.co * l.ci * 27), nchunk, l.cip, l.co, l.ci, wpart, cpart, m->g + l.off,
                               m->g + l.off + (long)l.co * l.ci * 27};
        if (q == 0) break;
        // data gradient, turned into the gradient entering layer q - 1
        ConvOut O{};
        if (q == 2 || q == 4 || q == 6) {
            O.yf = m->gtmp;
            launch_conv<CONV_F32>(m, n, V, l.co, l.cip, gb, m->Wf[q], O);
            k_pool_bwd<<<nblk((size_t)V * 2 * l.cip), 256, 0, m->stream>>>(B, 2 * n, l.cip, m->gtmp, m->gskip[q - 1],
                                                                           m->out[q - 1], gnext);
        } else if (q == 8 || q == 10 || q == 12) {
            // input channels: the upsampled output of layer q - 1, then the skip connection's
            const int C0u = m->L[q - 1].co;
            O.yf = m->gtmp;
            O.yf2 = m->gskip[skip_of(q)];
            O.c_lo = C0u;
            launch_conv<CONV_SPLIT>(m, n, V, l.co, l.cip, gb, m->Wf[q], O);
            k_up_bwd<<<nblk((size_t)V / 8 * C0u / 4), 256, 0, m->stream>>>(B, n / 2, C0u, m->gtmp, m->out[q - 1], gnext);
        } else {
            O.gate = m->out[q - 1];
            O.yb = gnext;
            launch_conv<CONV_GATE>(m, n, V, l.co, l.cip, gb, m->Wf[q], O);
        }
    }
    int blocks = 0;
    for (GradLayer &l : grads.l) {
        l.block0 = blocks;
        blocks += l.wblocks + l.co;
    }
    k_grad_final<<<blocks, 256, 0, m->stream>>>(grads);
}

void free_model(cps_model *m)
{
    if (!m) return;
    if (m->stream) (void)hipStreamSynchronize(m->stream);
    for (void *p : m->allocs) (void)hipFree(p);
    delete m;
}

}  // namespace

extern "C" {

int64_t cps_model_param_count(const cps_model_spec *spec)
{
    if (!spec) return -1;
    LayerInfo L[NLAYER];
    layer_table(spec->channels, spec->in_ch, L);
    return L[NLAYER - 1].off + (long)L[NLAYER - 1].co * L[NLAYER - 1].ci * 27 + L[NLAYER - 1].co + spec->channels[0] + 1;
}

int cps_model_create(cps_model **out, const cps_model_spec *spec, void *stream)
{
    if (!out || !spec || spec->struct_size != (int32_t)sizeof(cps_model_spec)) return CPS_EINVAL;
    if (spec->nc < 8 || spec->nc % 8 || spec->batch < 1 || spec->in_ch < 1 || spec->in_ch > 16) return CPS_EINVAL;
    for (int q = 0; q < 4; ++q)
        if (spec->channels[q] < 16 || spec->channels[q] % 16 || spec->channels[q] > 64) return CPS_EINVAL;
    if (spec->channels[0] > 16) return CPS_EINVAL;   // the head reduction holds 16 channels
    *out = nullptr;
    cps_model *m = new (std::nothrow) cps_model();
    if (!m) return CPS_ENOMEM;
    m->spec = *spec;
    m->stream = (hipStream_t)stream;
    try {
        nck(hipGetDevice(&m->device));
        layer_table(spec->channels, spec->in_ch, m->L);
        m->head_off = m->L[NLAYER - 1].off + (long)m->L[NLAYER - 1].co * m->L[NLAYER - 1].ci * 27 + m->L[NLAYER - 1].co;
        m->nparam = m->head_off + spec->channels[0] + 1;
        m->w = nalloc<float>(m, m->nparam);
        m->g = nalloc<float>(m, m->nparam);
        m->m1 = nalloc<float>(m, m->nparam);
        m->m2 = nalloc<float>(m, m->nparam);
        const int B = spec->batch, nc = spec->nc;
        size_t maxci = 0, maxco = 0;
        for (int q = 0; q < NLAYER; ++q) {
            LayerInfo &l = m->L[q];
            const int n = nc >> l.lvl;
            const size_t V = (size_t)B * n * n * n;
            m->Wk[q] = nalloc<bf16>(m, (size_t)l.co * 27 * l.cip);
            if (q > 0) m->Wf[q] = nalloc<bf16>(m, (size_t)l.cip * 27 * l.co);
            m->out[q] = nalloc<bf16>(m, V * l.co);
            if (q == 1 || q == 3 || q == 5) m->gskip[q] = nalloc<float>(m, V * l.co);
            if (q == 2 || q == 4 || q == 6) maxci = std::max(maxci, V * l.cip);
            if (q == 8 || q == 10 || q == 12) maxci = std::max(maxci, V * m->L[q - 1].co);
            maxco = std::max(maxco, V * l.co);
            // the chunk count for every batch size up to B (the chunk size depends on V)
            size_t part = 0;
            for (int bb = 1; bb <= B; ++bb) {
                const size_t Vb = (size_t)bb * n * n * n;
                const size_t wchunk = wgrad_chunk((int)Vb), nchunk = (Vb + wchunk - 1) / wchunk;
                part = std::max(part, nchunk * l.co * 27 * l.cip);
            }
            l.part = m->wpart_n;
            m->wpart_n += part;
        }
        for (int q = 0; q < NLAYER; ++q) {
            LayerInfo &l = m->L[q];
            const int n = nc >> l.lvl;
            const size_t V = (size_t)B * n * n * n;
            if (q == 0 || q == 2 || q == 4 || q == 6 || q == 8 || q == 10 || q == 12) {
                m->in[q] = nalloc<bf16>(m, V * l.cip);
                m->in_owned[q] = true;
            } else {
                m->in[q] = m->out[q - 1];
            }
        }
        m->gtmp = nalloc<float>(m, maxci);
        m->gb = nalloc<bf16>(m, maxco);
        m->gb2 = nalloc<bf16>(m, maxco);
        m->wpart = nalloc<float>(m, m->wpart_n);
        const size_t V0 = (size_t)B * nc * nc * nc;
        m->pred = nalloc<float>(m, V0);
        m->inp = nalloc<float>(m, (size_t)nc * nc * nc * spec->in_ch);   // one restricted problem
        m->lpart = nalloc<double>(m, std::max(2 * LOSS_BLOCKS, SCALE_BLOCKS));
        m->lossv = nalloc<double>(m, 2);
        m->sig = nalloc<double>(m, 1);
        m->hpart = nalloc<float>(m, HEAD_BLOCKS * 17);
        m->cpart = nalloc<float>(m, (size_t)NLAYER * COLSUM_PARTS * 64);   // channels are at most 64
        // He-normal initialisation from the spec's seed (host, deterministic)
        std::vector<float> h(m->nparam, 0.f);
        uint64_t st = spec->seed * 6364136223846793005ULL + 1442695040888963407ULL;
        auto unif = [&]() {
            st = st * 6364136223846793005ULL + 1442695040888963407ULL;
            return ((st >> 11) + 0.5) * (1.0 / 9007199254740992.0);
        };
        for (int q = 0; q < NLAYER; ++q) {
            const LayerInfo &l = m->L[q];
            double sd = std::sqrt(2.0 / (27.0 * l.ci));
            for (long e = 0; e < (long)l.co * l.ci * 27; ++e)
                h[l.off + e] = (float)(sd * std::sqrt(-2.0 * std::log(unif())) * std::cos(2.0 * M_PI * unif()));
        }
        for (int c = 0; c < spec->channels[0]; ++c)
            h[m->head_off + c] = (float)(std::sqrt(1.0 / spec->channels[0]) * (2.0 * unif() - 1.0));
        nck(hipMemcpyAsync(m->w, h.data(), sizeof(float) * m->nparam, hipMemcpyHostToDevice, m->stream));
        repack(m);
        nck(hipStreamSynchronize(m->stream));
    } catch (NetFail &f) {
        free_model(m);
        return f.code;
    }
    *out = m;
    return CPS_OK;
}

int cps_model_set_params(cps_model *m, const float *params, int64_t n)
{
    if (!m || !params || n != m->nparam) return CPS_EINVAL;
    try {
        nck(hipMemcpyAsync(m->w, params, sizeof(float) * n, hipMemcpyHostToDevice, m->stream));
        nck(hipMemsetAsync(m->m1, 0, sizeof(float) * n, m->stream));
        nck(hipMemsetAsync(m->m2, 0, sizeof(float) * n, m->stream));
        m->adam_t = 0;
        repack(m);
        nck(hipStreamSynchronize(m->stream));
    } catch (NetFail &f) {
        return f.code;
    }
    return CPS_OK;
}

int cps_model_get_params(cps_model *m, float *params, float *grads, int64_t n)
{
    if (!m || n != m->nparam) return CPS_EINVAL;
    try {
        if (params) nck(hipMemcpyAsync(params, m->w, sizeof(float) * n, hipMemcpyDeviceToHost, m->stream));
        if (grads) nck(hipMemcpyAsync(grads, m->g, sizeof(float) * n, hipMemcpyDeviceToHost, m->stream));
        nck(hipStreamSynchronize(m->stream));
    } catch (NetFail &f) {
        return f.code;
    }
    return CPS_OK;
}

int cps_model_forward(cps_model *m, const float *inputs, int32_t batch, float *pred)
{
    if (!m || !inputs || !pred || batch < 1 || batch > m->spec.batch) return CPS_EINVAL;
    try {
        forget_errors();
        const size_t n3 = (size_t)m->spec.nc * m->spec.nc * m->spec.nc, ci = m->spec.in_ch;
        const bool in_place = cps::device_array(pred, batch * n3 * sizeof(float), m->device);
        forward(m, batch, readable(m, inputs, batch * n3 * ci, 0, m->spec.batch * n3 * ci), in_place ? pred : m->pred);
        nck(hipGetLastError());
        if (!in_place) nck(hipMemcpyAsync(pred, m->pred, batch * n3 * sizeof(float), hipMemcpyDefault, m->stream));
        nck(hipStreamSynchronize(m->stream));
    } catch (NetFail &f) {
        return f.code;
    }
    return CPS_OK;
}

int cps_model_train_step(cps_model *m, const float *inputs, const float *target, const float *mask, int32_t batch,
                         float lr, int32_t update, double *loss_out)
{
    if (!m || !inputs || !target || batch < 1 || batch > m->spec.batch) return CPS_EINVAL;
    try {
        forget_errors();
        const size_t n3 = (size_t)m->spec.nc * m->spec.nc * m->spec.nc, ci = m->spec.in_ch, most = m->spec.batch * n3;
        forward(m, batch, readable(m, inputs, batch * n3 * ci, 0, most * ci), m->pred);
        backward(m, batch, readable(m, target, batch * n3, 1, most), readable(m, mask, batch * n3, 2, most));
        if (update) {
            m->adam_t++;
            const float b1 = 0.9f, b2 = 0.999f;
            float c1 = 1.f - std::pow(b1, (float)m->adam_t), c2 = 1.f - std::pow(b2, (float)m->adam_t);
            k_adam<<<nblk(m->nparam), 256, 0, m->stream>>>(m->nparam, m->w, m->g, m->m1, m->m2, lr, b1, b2, 1e-8f, c1, c2);
            repack(m);
        }
        nck(hipGetLastError());
        double lv[2];
        nck(hipMemcpyAsync(lv, m->lossv, sizeof(double) * 2, hipMemcpyDeviceToHost, m->stream));
        nck(hipStreamSynchronize(m->stream));
        if (loss_out) *loss_out = lv[0];
    } catch (NetFail &f) {
        return f.code;
    }
    return CPS_OK;
}

int cps_model_restrict(cps_model *m, cps_solver *s, const double *u, float *inputs, float *target, double *sigma)
{
    if (!m || !s || !inputs) return CPS_EINVAL;
    try {
        return restrict_into(m, s, u, inputs, target, sigma, m->lpart, m->sig);
    } catch (NetFail &f_) {
        return f_.code;
    }
}

int cps_model_restrict_noalloc(cps_model *m, cps_solver *s, const double *u, float *inputs, float *target,
                               double *sigma)
{
    if (!m || !s || !inputs) return CPS_EINVAL;
    try {
        double *sp = scratch_address(m->device);
        return restrict_into(m, s, u, inputs, target, sigma, sp, sp + SCALE_BLOCKS);
    } catch (NetFail &f_) {
        return f_.code;
    }
}

int cps_model_predict(cps_model *m, cps_solver *s, double *u0)
{
    if (!m || !s || !u0) return CPS_EINVAL;
    const double *phi, *g, *f;
    int nx, ny, nz;
    void *sst;
    cps_internal_fields(s, &phi, &g, &f, &nx, &ny, &nz, &sst);
    const int nc = m->spec.nc;
    try {
        int rc = cps_model_restrict(m, s, nullptr, m->inp, nullptr, nullptr);
        if (rc) return rc;
        forward(m, 1, m->inp, m->pred);
        size_t nn = (size_t)nx * ny * nz;
        k_prolong<<<dim3(nblk((size_t)nx), (unsigned)ny, (unsigned)nz), 256, 0, m->stream>>>(nx, ny, nz, nc, m->pred,
                                                                                            m->sig, u0);
        nck(hipStreamSynchronize(m->stream));
    } catch (NetFail &f_) {
        return f_.code;
    }
    return CPS_OK;
}

int cps_model_predict_fields(cps_model *m, int32_t nx, int32_t ny, int32_t nz, const double *phi, const double *g,
                             const double *f, double *u0, void *stream)
{
    if (!m || !phi || !g || !f || !u0) return CPS_EINVAL;
    // the call's kernels go to `stream`; the model's own stream is restored on every return
    struct Restore {
        cps_model *m;
        hipStream_t st;
        ~Restore() { m->stream = st; }
    } restore{m, m->stream};
    if (stream) m->stream = (hipStream_t)stream;
    const int nc = m->spec.nc;
    try {
        int rc = restrict_fields(m, nx, ny, nz, phi, g, f, nullptr, m->inp, nullptr, nullptr, m->lpart, m->sig, false);
        if (rc) return rc;
        forward(m, 1, m->inp, m->pred);
        k_prolong<<<dim3(nblk((size_t)nx), (unsigned)ny, (unsigned)nz), 256, 0, m->stream>>>(nx, ny, nz, nc, m->pred,
                                                                                            m->sig, u0);
        nck(hipGetLastError());
    } catch (NetFail &f_) {
        return f_.code;
    }
    return CPS_OK;
}

namespace {

// File layout: 8-byte magic, the spec, nparam (long), then the FP32 weights; a checkpoint
// ("CPSNET02") adds the Adam step count (int64) and the two FP32 moment vectors.
int write_model(cps_model *m, const char *path, bool with_optimizer)
{
    if (!m || !path) return CPS_EINVAL;
    const size_t n = (size_t)m->nparam;
    std::vector<float> h(with_optimizer ? 3 * n : n);
    try {
        nck(hipMemcpyAsync(h.data(), m->w, sizeof(float) * n, hipMemcpyDeviceToHost, m->stream));
        if (with_optimizer) {
            nck(hipMemcpyAsync(h.data() + n, m->m1, sizeof(float) * n, hipMemcpyDeviceToHost, m->stream));
            nck(hipMemcpyAsync(h.data() + 2 * n, m->m2, sizeof(float) * n, hipMemcpyDeviceToHost, m->stream));
        }
        nck(hipStreamSynchronize(m->stream));
    } catch (NetFail &f) {
        return f.code;
    }
    FILE *fp = std::fopen(path, "wb");
    if (!fp) return CPS_EINVAL;
    const char *magic = with_optimizer ? "CPSNET02" : "CPSNET01";
    const int64_t t = m->adam_t;
    bool ok = std::fwrite(magic, 1, 8, fp) == 8 && std::fwrite(&m->spec, sizeof(m->spec), 1, fp) == 1 &&
              std::fwrite(&m->nparam, sizeof(m->nparam), 1, fp) == 1 &&
              (!with_optimizer || std::fwrite(&t, sizeof(t), 1, fp) == 1) &&
              std::fwrite(h.data(), sizeof(float), h.size(), fp) == h.size();
    ok = (std::fclose(fp) == 0) && ok;
    return ok ? CPS_OK : CPS_EINVAL;
}

}  // namespace

int cps_model_save(cps_model *m, const char *path) { return write_model(m, path, false); }

int cps_model_save_checkpoint(cps_model *m, const char *path) { return write_model(m, path, true); }

int cps_model_load(cps_model *m, const char *path)
{
    if (!m || !path) return CPS_EINVAL;
    FILE *fp = std::fopen(path, "rb");
    if (!fp) return CPS_EINVAL;
    char magic[8];
    cps_model_spec sp;
    long np = 0;
    int64_t t = 0;
    bool ok = std::fread(magic, 1, 8, fp) == 8 && std::fread(&sp, sizeof(sp), 1, fp) == 1 &&
              std::fread(&np, sizeof(np), 1, fp) == 1 && np == m->nparam;
    const bool ckpt = ok && std::memcmp(magic, "CPSNET02", 8) == 0;
    ok = ok && (ckpt || std::memcmp(magic, "CPSNET01", 8) == 0);
    if (ok && ckpt) ok = std::fread(&t, sizeof(t), 1, fp) == 1 && t >= 0 && t <= (int64_t)INT32_MAX;
    std::vector<float> h;
    if (ok) {
        h.resize(ckpt ? 3 * (size_t)np : (size_t)np);
        ok = std::fread(h.data(), sizeof(float), h.size(), fp) == h.size();
    }
    std::fclose(fp);
    if (!ok) return CPS_EINVAL;
    // the weights (and a fresh optimiser); a checkpoint then restores Adam's moments and step
    const int rc = cps_model_set_params(m, h.data(), np);
    if (rc != CPS_OK || !ckpt) return rc;
    try {
        nck(hipMemcpyAsync(m->m1, h.data() + np, sizeof(float) * np, hipMemcpyHostToDevice, m->stream));
        nck(hipMemcpyAsync(m->m2, h.data() + 2 * np, sizeof(float) * np, hipMemcpyHostToDevice, m->stream));
        nck(hipStreamSynchronize(m->stream));
    } catch (NetFail &f) {
        return f.code;
    }
    m->adam_t = (int)t;
    return CPS_OK;
}

void cps_model_destroy(cps_model *m) { free_model(m); }

}  // extern "C"
