// Learned pressure-stage correction: a 3-D convolutional network (four
// zero-padded 3x3x3 convolutions, channels 2 -> 16 -> 16 -> 16 -> 1, biases,
// ReLU after the first three) trained on pairs of pressure residual and the
// error one AMG V-cycle leaves.  Forward and backward passes run on the
// matrix cores: BF16 operands, FP32 accumulation (v_mfma_f32_16x16x32_bf16,
// lane l holding A[l % 16][8 (l / 16) + j], B[8 (l / 16) + j][l % 16] for
// j < 8, and receiving C[4 (l / 16) + j][l % 16] for j < 4).
//
// Convolution as an implicit GEMM.  A workgroup owns output tiles of 16 (x) by
// 4 (y) by 4 (z) voxels = 16 rows of 16 voxels; its four wavefronts take four
// rows each.  The input halo (18 x 6 x 6 voxels, BF16) is staged in LDS, the
// layer's weights stay in registers.  For one row and one tap the product is
// D[n][i] = sum_k W[t][n][k] X[i + off(t)][k] with n the output channel, i the
// voxel of the row and k the input channel, with the weights as the A operand
// and the shifted row as the B operand, so that lane l ends with output
// channels 4(l/16)..4(l/16)+3 of voxel l%16 and stores them as one 8-byte
// write.  One 16x16x32 MFMA covers two taps of 16 input channels (lane groups
// 0-1 the first tap, 2-3 the second; 27 taps padded to 28 with a zero one): 14
// per row.  The first layer has 2 input channels (padded to 4): one MFMA covers
// eight taps, each lane group two of them (27 taps padded to 32).
//
// Backward: the input gradient of a layer is the same convolution with the
// kernel flipped and transposed (dX[u][c] = sum_t sum_o dZ[u - off(t)][o]
// W[t][c][o]), masked by the ReLU of the layer below; the weight gradient
// dW[t][c][o] = sum_v X[v + off(t)][c] dZ[v][o] is an MFMA reduction over the
// voxels of each tile (32 voxels, two rows, per MFMA), combined across
// workgroups in a fixed order.
#include <cstring>
#include <type_traits>
#include "bo_nn.hpp"
#include "bo_cpr.hpp"

namespace bo {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// eight BF16 values (16 bytes) as an MFMA operand
__device__ __forceinline__ v8bf bf8(uint4 u) { return __builtin_bit_cast(v8bf, u); }

constexpr int TX = 16, TY = 4, TZ = 4;
constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2;
constexpr int HV = HX * HY * HZ;      // halo voxels of a tile
constexpr int TV = TX * TY * TZ;      // voxels of a tile
enum { MODE_ACT = 0, MODE_OUT = 1, MODE_GRAD = 2 };

// FP32 -> BF16 (round to nearest even; values are finite) and back
__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint32_t h) { return __uint_as_float(h << 16); }

struct TileXY {
    int b, z0, y0, x0;
};
__device__ __forceinline__ TileXY tile_of(const Vol &V, int tile) {
    int ntx = (V.nx + TX - 1) / TX, nty = (V.ny + TY - 1) / TY, ntz = (V.nz + TZ - 1) / TZ;
    TileXY T;
    T.x0 = (tile % ntx) * TX;
    tile /= ntx;
    T.y0 = (tile % nty) * TY;
    tile /= nty;
    T.z0 = (tile % ntz) * TZ;
    T.b = tile / ntz;
    return T;
}
inline long long tiles_of(const Vol &V) {
    return (long long)((V.nx + TX - 1) / TX) * ((V.ny + TY - 1) / TY) * ((V.nz + TZ - 1) / TZ) * V.nb;
}
__device__ __forceinline__ long long voxel(const Vol &V, int b, int z, int y, int x) {
    return (((long long)b * V.nz + z) * V.ny + y) * V.nx + x;
}

__device__ __forceinline__ int halo_index(int z, int y, int x) { return (z * HY + y) * HX + x; }

// The tiles a workgroup visits: each XCD owns one contiguous range of tiles
// (workgroups are dealt to the eight XCDs round-robin), so the halos that
// neighbouring tiles share are read from that XCD's L2.  The grid is a
// multiple of 8.
struct TileRange {
    int first, last, step;
};
__device__ __forceinline__ TileRange tiles_of_block(int ntiles) {
    const int x = blockIdx.x % 8, q = blockIdx.x / 8;
    const int per = ntiles / 8, rem = ntiles % 8;
    const int base = x * per + min(x, rem);
    return {base + q, base + per + (x < rem ? 1 : 0), (int)gridDim.x / 8};
}

// Convolution of a CIN-channel input to 16 output channels.  W: [taps][16][CIN]
// BF16 (27 taps and zero ones up to 28 (CIN = 16) or 32 (CIN = 4)).
//   MODE_ACT:  out = BF16(ReLU(acc + bias))              -> act_out [v][16]
//   MODE_OUT:  y = acc[channel 0] + bias[0]              -> y_out [v] (FP32), and y_copy [v] unless NULL
//   MODE_GRAD: out = BF16(acc) where mask[v][n] > 0, else 0 -> act_out [v][16]
// Bound by LDS reads (14 KB per row of 16 voxels, 22 us for 2M voxels) and by
// the activations' traffic (64 B per voxel, 25 us), not by the matrix cores
// (11 us).  The weights therefore stay in registers over all tiles of a
// workgroup, the halo is kept as two planes of 8 channels (16 B per voxel: the
// 16 lanes of a row read 256 contiguous bytes, no bank conflict), the tap
// offsets are four registers and constants, and four rows' accumulators run
// interleaved; registers stay at 128, four workgroups per CU.  16 -> 16
// channels over 2M voxels: 132 us with weights and offsets taken per row from
// LDS, 49 us now (2.6 TB/s of the 128 B per voxel).
template <int CIN, int MODE>
__global__ void __launch_bounds__(256, 4) k_nn_conv(Vol V, int ntiles, const uint16_t *__restrict__ in,
                                                 const uint16_t *__restrict__ W, const float *__restrict__ bias,
                                                 const uint16_t *__restrict__ mask, uint16_t *__restrict__ act_out,
                                                 float *__restrict__ y_out, float *__restrict__ y_copy) {
    typedef typename std::conditional<CIN == 16, uint4, uint2>::type Vec;  // one plane's part of a voxel
    constexpr int NP = CIN == 16 ? 2 : 1;                                  // planes
    constexpr int NLD = (HV * NP + 255) / 256;
    constexpr int NOP = CIN == 16 ? 14 : 4;                                // MFMAs per row
    __shared__ __align__(16) Vec xs[NP * HV];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int i = lane % 16, g = lane / 16;
    // A operands and LDS offsets of the taps.  CIN = 16: k = 8g + j is tap
    // 2 tp + g / 2, input channel 8 (g % 2) + j.  CIN = 4: k = 8g + 4h + j is
    // tap 8q + 2g + h, input channel j.  Taps past 26 have zero weights.
    // For CIN = 16 the second tap of a pair is 1 voxel, one row less 2 or one
    // plane less 2 rows and 2 voxels further on (0 for the padding tap): four
    // lane offsets, the rest are constants.
    v8bf wa[NOP];
    int off[NOP], off2[NOP], base[4];
    base[0] = wave * HY * HX + i + (g & 1) * HV;
    base[1] = base[0] + (g >> 1);
    base[2] = base[0] + (g >> 1) * (HX - 2);
    base[3] = base[0] + (g >> 1) * (HX * HY - 2 * HX - 2);
#pragma unroll
    for (int q = 0; q < NOP; q++) {
        const int t0 = CIN == 16 ? 2 * q + (g >> 1) : 8 * q + 2 * g;
        const int ta = min(t0, 26), tb = min(t0 + 1, 26);
        const int row0 = wave * HY * HX + i;
        if (CIN == 16) {
            wa[q] = bf8(*(const uint4 *)(W + (t0 * 16 + i) * 16 + 8 * (g & 1)));
        } else {
            off[q] = row0 + halo_index(ta / 9, (ta / 3) % 3, ta % 3);
            off2[q] = row0 + halo_index(tb / 9, (tb / 3) % 3, tb % 3);
            const uint2 a = *(const uint2 *)(W + (t0 * 16 + i) * 4), b = *(const uint2 *)(W + ((t0 + 1) * 16 + i) * 4);
            wa[q] = bf8(make_uint4(a.x, a.y, b.x, b.y));
        }
    }
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (MODE != MODE_GRAD)
        for (int j = 0; j < 4; j++) bv[j] = (MODE == MODE_OUT && 4 * g + j > 0) ? 0.f : bias[4 * g + j];
    const TileRange R = tiles_of_block(ntiles);
    for (int tile = R.first; tile < R.last; tile += R.step) {
        const TileXY T = tile_of(V, tile);
        // the halo (zero outside the volume), every load in flight at once; the
        // other workgroups of the CU cover the wait (keeping the next tile's
        // halo in registers during the products costs more occupancy than it
        // hides: 72 against 49 us at 2M voxels)
        Vec ld[NLD];
#pragma unroll
        for (int u = 0; u < NLD; u++) {
            const int q = threadIdx.x + 256 * u;
            const int hv = q / NP, p = q % NP;
            const int hx = hv % HX, hy = (hv / HX) % HY, hz = hv / (HX * HY);
            const int x = T.x0 + hx - 1, y = T.y0 + hy - 1, z = T.z0 + hz - 1;
            Vec val = {};
            if (q < NP * HV && x >= 0 && x < V.nx && y >= 0 && y < V.ny && z >= 0 && z < V.nz)
                val = ((const Vec *)in)[voxel(V, T.b, z, y, x) * NP + p];
            ld[u] = val;
        }
        __syncthreads();  // the previous tile's reads
#pragma unroll
        for (int u = 0; u < NLD; u++) {
            const int q = threadIdx.x + 256 * u;
            if (q < NP * HV) xs[(q % NP) * HV + q / NP] = ld[u];
        }
        __syncthreads();
        v4f acc[4];
#pragma unroll
        for (int rr = 0; rr < 4; rr++) acc[rr] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < NOP; q++)
#pragma unroll
            for (int rr = 0; rr < 4; rr++) {
                v8bf b;
                if constexpr (CIN == 16) {
                    constexpr int ahead[14] = {1, 2, 1, 1, 3, 1, 1, 2, 1, 1, 2, 1, 1, 0};
                    const int t = 2 * q;
                    b = bf8(xs[base[ahead[q]] + halo_index(t / 9, (t / 3) % 3, t % 3) + rr * HX]);
                } else {
                    const uint2 u = xs[off[q] + rr * HX], w = xs[off2[q] + rr * HX];
                    b = bf8(make_uint4(u.x, u.y, w.x, w.y));
                }
                acc[rr] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[q], b, acc[rr], 0, 0, 0);
            }
        const int x = T.x0 + i, z = T.z0 + wave;
        if (x >= V.nx || z >= V.nz) continue;
        const long long v0 = voxel(V, T.b, z, T.y0, x);
#pragma unroll
        for (int rr = 0; rr < 4; rr++) {
            if (T.y0 + rr >= V.ny) break;
            const long long v = v0 + (long long)rr * V.nx;
            if (MODE == MODE_OUT) {
                if (g == 0) {
                    const float y = acc[rr][0] + bv[0];
                    y_out[v] = y;
                    if (y_copy) y_copy[v] = y;
                }
            } else {
                uint16_t o[4];
                if (MODE == MODE_ACT) {
                    for (int j = 0; j < 4; j++) o[j] = to_bf16(fmaxf(acc[rr][j] + bv[j], 0.f));
                } else {
                    uint2 mk = *(const uint2 *)(mask + v * 16 + 4 * g);
                    uint32_t mw[4] = {mk.x & 0xFFFFu, mk.x >> 16, mk.y & 0xFFFFu, mk.y >> 16};
                    for (int j = 0; j < 4; j++) o[j] = (mw[j] & 0x7FFFu) ? to_bf16(acc[rr][j]) : (uint16_t)0;
                }
                *(uint2 *)(act_out + v * 16 + 4 * g) =
                    make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
            }
        }
    }
}

// two voxels' channel pairs (a: channels c, c+1 of the first voxel, b: of the
// second) as one word per channel
__device__ __forceinline__ uint32_t chan_lo(uint32_t a, uint32_t b) { return (a & 0xFFFFu) | (b << 16); }
__device__ __forceinline__ uint32_t chan_hi(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xFFFF0000u); }

// voxel pair (a, b) into one plane per channel (S 16-bit words apart): eight
// channels, or the N used ones of a 4-channel voxel
template <int S, int N>
__device__ __forceinline__ void put_pair(uint32_t *o, const uint4 &a, const uint4 &b) {
    constexpr int P = S / 2;
    o[0 * P] = chan_lo(a.x, b.x); o[1 * P] = chan_hi(a.x, b.x);
    o[2 * P] = chan_lo(a.y, b.y); o[3 * P] = chan_hi(a.y, b.y);
    o[4 * P] = chan_lo(a.z, b.z); o[5 * P] = chan_hi(a.z, b.z);
    o[6 * P] = chan_lo(a.w, b.w); o[7 * P] = chan_hi(a.w, b.w);
}
template <int S, int N>
__device__ __forceinline__ void put_pair(uint32_t *o, const uint2 &a, const uint2 &b) {
    o[0] = chan_lo(a.x, b.x);
    if (N > 1) o[S / 2] = chan_hi(a.x, b.x);
}

// Weight and bias gradients of one layer: dW[t][c][o] = sum_v X[v+off(t)][c]
// dZ[v][o], db[o] = sum_v dZ[v][o], with X the layer's input (CIN channels
// stored, CI used) and dZ its output gradient (COUT stored, CO used; channels
// past CO are zero).  The products reduce over voxels, so both operands need 8
// consecutive voxels of one channel per lane: the tile is transposed to one
// plane per channel on its way into LDS (two voxels per 32-bit word).  A lane
// then reads the ten voxels its three x-shifts cover as one 16-byte and one
// 4-byte read and forms the middle shift with four funnel shifts; the plane
// strides (1744 and 528 bytes) put the 16 channels of a read in distinct
// banks.  Six wavefronts: z-shift (3) x half of the tile's rows (2), nine
// 16x16 accumulators each; the halves meet in LDS once per workgroup, which
// writes its sums to part[workgroup][gradient layout] (kNnPartStride apart).
// Bound by the staging (LDS writes and the loads' latency; the next tile's
// loads are in flight during the products).  16 -> 16 channels at 524288
// voxels: 78 us with 16-bit LDS gathers and 27 accumulators per wavefront,
// 18 us now.
template <int CIN, int CI, int COUT, int CO>
__global__ void __launch_bounds__(384) k_nn_wgrad(Vol V, int ntiles, const uint16_t *__restrict__ X,
                                                  const uint16_t *__restrict__ dZ, float *__restrict__ part) {
    constexpr int PX = 24;            // halo row pitch, 16-bit words
    constexpr int XS = 872;           // plane strides, 16-bit words
    constexpr int DS = 264;
    constexpr int XW = 16 * XS / 2, DW = 16 * DS / 2;
    constexpr int CMB = 3 * 40 * 64;  // the combination at the end, 32-bit words
    __shared__ __align__(16) uint32_t sm[XW + DW > CMB ? XW + DW : CMB];
    uint16_t *xs = (uint16_t *)sm, *ds = (uint16_t *)(sm + XW);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int c = lane % 16, g = lane / 16;   // A: output channel o = c; B: input channel = c
    const int dzi = wave % 3, half = wave / 3;
    // lanes past the used channels repeat a used one; their sums are dropped
    const uint16_t *xb = xs + (c < CI ? c : 0) * XS + 8 * (g & 1);
    const uint16_t *db = ds + (c < CO ? c : 0) * DS + 8 * (g & 1);
    v4f acc[9], accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; t++) acc[t] = (v4f){0.f, 0.f, 0.f, 0.f};
    const v8bf ones = bf8(make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
    const TileRange R = tiles_of_block(ntiles);
    // voxel pairs of the X halo and of dZ per thread: (pair, group of 8 (16
    // stored channels) or 2 channels); the next tile's are in flight while the
    // current one is worked on
    typedef typename std::conditional<CIN == 16, uint4, uint2>::type XVec;
    typedef typename std::conditional<COUT == 16, uint4, uint2>::type DVec;
    constexpr int XG = CIN == 16 ? 2 : 1, DG = COUT == 16 ? 2 : 1;
    constexpr int NX = (HV / 2 * XG + 383) / 384, ND = (TV / 2 * DG + 383) / 384;
    XVec xa[NX], xc[NX];
    DVec da[ND], dc[ND];
    auto load = [&](const TileXY &T) {
#pragma unroll
        for (int u = 0; u < NX; u++) {
            const int q = threadIdx.x + 384 * u;
            const int h = q % XG, pr = q / XG;
            const int px = pr % (HX / 2), hy = (pr / (HX / 2)) % HY, hz = pr / (HX / 2 * HY);
            const int x = T.x0 + 2 * px - 1, y = T.y0 + hy - 1, z = T.z0 + hz - 1;
            const bool in = q < HV / 2 * XG && y >= 0 && y < V.ny && z >= 0 && z < V.nz;
            const long long v = voxel(V, T.b, z, y, x);
            XVec a = {}, b = {};
            if (in && x >= 0 && x < V.nx) a = ((const XVec *)X)[XG * v + h];
            if (in && x + 1 < V.nx) b = ((const XVec *)X)[XG * (v + 1) + h];
            xa[u] = a;
            xc[u] = b;
        }
#pragma unroll
        for (int u = 0; u < ND; u++) {
            const int q = threadIdx.x + 384 * u;
            const int h = q % DG, pr = q / DG;
            const int px = pr % (TX / 2), ty = (pr / (TX / 2)) % TY, tz = pr / (TX / 2 * TY);
            const int x = T.x0 + 2 * px, y = T.y0 + ty, z = T.z0 + tz;
            const bool in = q < TV / 2 * DG && y < V.ny && z < V.nz;
            const long long v = voxel(V, T.b, z, y, x);
            DVec a = {}, b = {};
            if (in && x < V.nx) a = ((const DVec *)dZ)[DG * v + h];
            if (in && x + 1 < V.nx) b = ((const DVec *)dZ)[DG * (v + 1) + h];
            da[u] = a;
            dc[u] = b;
        }
    };
    if (R.first < R.last) load(tile_of(V, R.first));
    for (int tile = R.first; tile < R.last; tile += R.step) {
        __syncthreads();  // the previous tile's reads
#pragma unroll
        for (int u = 0; u < NX; u++) {
            const int q = threadIdx.x + 384 * u;
            const int h = q % XG, pr = q / XG;
            const int px = pr % (HX / 2), row = pr / (HX / 2);
            if (q < HV / 2 * XG) put_pair<XS, 2>((uint32_t *)xs + row * (PX / 2) + px + 8 * h * (XS / 2), xa[u], xc[u]);
        }
#pragma unroll
        for (int u = 0; u < ND; u++) {
            const int q = threadIdx.x + 384 * u;
            const int h = q % DG, pr = q / DG;
            if (q < TV / 2 * DG) put_pair<DS, 1>((uint32_t *)ds + pr + 8 * h * (DS / 2), da[u], dc[u]);
        }
        __syncthreads();
        if (tile + R.step < R.last) load(tile_of(V, tile + R.step));
        // two rows of 16 voxels per MFMA: k = 8g + j is voxel 8 (g % 2) + j of
        // row 2s + g / 2
#pragma unroll
        for (int ss = 0; ss < 4; ss++) {
            const int r = 2 * (4 * half + ss) + (g >> 1);
            const int ry = r % TY, rz = r / TY;
            const v8bf a = bf8(*(const uint4 *)(db + r * TX));
            if (dzi == 1) accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, accb, 0, 0, 0);
#pragma unroll
            for (int dy = 0; dy < 3; dy++) {
                const uint16_t *p = xb + ((rz + dzi) * HY + ry + dy) * PX;
                const uint4 w = *(const uint4 *)p;
                const uint32_t w4 = *(const uint32_t *)(p + 8);
                const uint4 m =
                    make_uint4(__builtin_amdgcn_alignbit(w.y, w.x, 16), __builtin_amdgcn_alignbit(w.z, w.y, 16),
                               __builtin_amdgcn_alignbit(w.w, w.z, 16), __builtin_amdgcn_alignbit(w4, w.w, 16));
                acc[3 * dy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bf8(w), acc[3 * dy], 0, 0, 0);
                acc[3 * dy + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bf8(m), acc[3 * dy + 1], 0, 0, 0);
                acc[3 * dy + 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bf8(make_uint4(w.y, w.z, w.w, w4)),
                                                                          acc[3 * dy + 2], 0, 0, 0);
            }
        }
    }
    // the two halves of the rows
    __syncthreads();
    float *cmb = (float *)sm + dzi * 40 * 64 + lane;
    if (half == 1) {
#pragma unroll
        for (int t = 0; t < 9; t++)
            for (int j = 0; j < 4; j++) cmb[(4 * t + j) * 64] = acc[t][j];
        for (int j = 0; j < 4; j++) cmb[(36 + j) * 64] = accb[j];
    }
    __syncthreads();
    if (half == 1) return;
    // D_t[o = 4g+j][c]
    float *out = part + (size_t)blockIdx.x * kNnPartStride;
#pragma unroll
    for (int t = 0; t < 9; t++)
        for (int j = 0; j < 4; j++) {
            const int o = 4 * g + j;
            if (c < CI && o < CO) out[((dzi * 9 + t) * CI + c) * CO + o] = acc[t][j] + cmb[(4 * t + j) * 64];
        }
    if (dzi == 1 && c == 0)   // every column holds the same sum
        for (int j = 0; j < 4; j++)
            if (4 * g + j < CO) out[27 * CI * CO + 4 * g + j] = accb[j] + cmb[(36 + j) * 64];
}

// The workgroups' gradients summed in a fixed order, all layers at once: 64
// parameters per workgroup, eight wavefronts taking every eighth part each.
// Bound by reading the parts once (15169 floats per workgroup of k_nn_wgrad);
// one thread per parameter over 1024 parts took 271 us per layer, all four
// layers take 7 us now.
__global__ void __launch_bounds__(512) k_nn_wgrad_reduce(int nparts, const float *__restrict__ part,
                                                         float *__restrict__ grad) {
    __shared__ double red[8][64];
    const int l = threadIdx.x % 64, w = threadIdx.x / 64;
    const int e = blockIdx.x * 64 + l;
    double s = 0.0;
    if (e < kNnParams)
#pragma unroll 8
        for (int p = w; p < nparts; p += 8) s += (double)part[(size_t)p * kNnPartStride + e];
    red[w][l] = s;
    __syncthreads();
    if (w != 0 || e >= kNnParams) return;
    for (int q = 1; q < 8; q++) s += red[q][l];
    grad[e] = (float)s;
}

// network input from FP32 pairs of channels [v][2] -> BF16 [v][4]
__global__ void k_nn_input(long long nv, const float *__restrict__ in, uint16_t *__restrict__ x) {
    long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    uint32_t h0 = to_bf16(in[2 * v]), h1 = to_bf16(in[2 * v + 1]);
    *(uint2 *)(x + 4 * v) = make_uint2(h0 | (h1 << 16), 0u);
}

// output gradient of the mean squared error: dZ4 = BF16(2 (y - t) / M) in a
// 4-channel tensor; partial sums of (y - t)^2 per block
__global__ void __launch_bounds__(256) k_nn_loss(long long nv, const float *__restrict__ y,
                                                 const float *__restrict__ tgt, float scale,
                                                 uint16_t *__restrict__ dz, double *__restrict__ lpart) {
    __shared__ double red[256];
    long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    double sq = 0.0;
    if (v < nv) {
        float d = y[v] - tgt[v];
        sq = (double)d * d;
        *(uint2 *)(dz + 4 * v) = make_uint2((uint32_t)to_bf16(d * scale), 0u);
    }
    red[threadIdx.x] = sq;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) lpart[blockIdx.x] = red[0];
}

// the partial sums of the loss in a fixed order, one workgroup (118 us for
// 2048 partial sums by one thread)
__global__ void __launch_bounds__(kBlock) k_nn_loss_final(int nparts, const double *__restrict__ lpart, double inv_m,
                                                          double *__restrict__ loss) {
    __shared__ double red[kBlock];
    double s = 0.0;
#pragma unroll 4
    for (int p = threadIdx.x; p < nparts; p += kBlock) s += lpart[p];
    s = block_sum(s, red);
    if (threadIdx.x == 0) *loss = s * inv_m;
}

// A_pp-weighted loss: R = A (y - t) on the voxels whose six neighbours lie in
// the volume (0 elsewhere), coef [7][voxels] in slot order (-z, -y, -x, self,
// +x, +y, +z); partial sums of R^2 per block
__global__ void __launch_bounds__(256) k_nn_wres(Vol V, const float *__restrict__ coef, const float *__restrict__ y,
                                                 const float *__restrict__ tgt, float *__restrict__ R,
                                                 double *__restrict__ lpart) {
    __shared__ double red[256];
    const long long nv = V.voxels();
    const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    double sq = 0.0;
    if (v < nv) {
        const int x = (int)(v % V.nx), yy = (int)((v / V.nx) % V.ny), z = (int)((v / ((long long)V.nx * V.ny)) % V.nz);
        float r = 0.f;
        if (x > 0 && x < V.nx - 1 && yy > 0 && yy < V.ny - 1 && z > 0 && z < V.nz - 1) {
            const long long sx = 1, sy = V.nx, sz = (long long)V.nx * V.ny;
            const long long nb[7] = {v - sz, v - sy, v - sx, v, v + sx, v + sy, v + sz};
            double acc = 0.0;
            for (int q = 0; q < 7; q++)
                acc += (double)coef[(size_t)q * nv + v] * (double)(y[nb[q]] - tgt[nb[q]]);
            r = (float)acc;
        }
        R[v] = r;
        sq = (double)r * r;
    }
    red[threadIdx.x] = sq;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) lpart[blockIdx.x] = red[0];
}

// output gradient of the weighted loss: dZ4 = BF16(scale (A^T R)) in a
// 4-channel tensor, (A^T R)_j = sum over the cells i whose slot q couples to
// j of coef[q][i] R_i
__global__ void k_nn_wout(Vol V, const float *__restrict__ coef, const float *__restrict__ R, float scale,
                          uint16_t *__restrict__ dz) {
    const long long nv = V.voxels();
    const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nv) return;
    const int x = (int)(j % V.nx), yy = (int)((j / V.nx) % V.ny), z = (int)((j / ((long long)V.nx * V.ny)) % V.nz);
    const long long sx = 1, sy = V.nx, sz = (long long)V.nx * V.ny;
    // cell i = j - off(q): slot q of i points at j
    const bool in[7] = {z < V.nz - 1, yy < V.ny - 1, x < V.nx - 1, true, x > 0, yy > 0, z > 0};
    const long long src[7] = {j + sz, j + sy, j + sx, j, j - sx, j - sy, j - sz};
    double g = 0.0;
    for (int q = 0; q < 7; q++)
        if (in[q]) g += (double)coef[(size_t)q * nv + src[q]] * (double)R[src[q]];
    *(uint2 *)(dz + 4 * j) = make_uint2((uint32_t)to_bf16((float)(scale * g)), 0u);
}

// where parameter e of the flat layout stands in the packed BF16 weights
struct PackedNet {
    uint16_t *wf[kNnLayers], *wb[kNnLayers];
};

// Adam, and the BF16 copies of the updated weights in the layouts of k_nn_pack
// (each weight has one place in either; the padding stays zero)
__global__ void k_nn_adam(int n, float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                          float *__restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2,
                          PackedNet P) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    float gi = g[e];
    float mi = b1 * m[e] + (1.f - b1) * gi;
    float vi = b2 * v[e] + (1.f - b2) * gi * gi;
    m[e] = mi;
    v[e] = vi;
    const float wn = w[e] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[e] = wn;
    const uint16_t h = to_bf16(wn);
    int off = 0;
#pragma unroll
    for (int l = 0; l < kNnLayers; l++) {
        constexpr int chan[kNnLayers + 1] = {2, 16, 16, 16, 1};
        const int ci = chan[l], co = chan[l + 1], nw = 27 * ci * co;
        const int q = e - off;
        if (q >= 0 && q < nw) {
            const int t = q / (ci * co), k = (q / co) % ci, o = q % co;
            const int kf = l == 0 ? 4 : 16, kb = l == kNnLayers - 1 ? 4 : 16;
            P.wf[l][(t * 16 + o) * kf + k] = h;
            if (l > 0) P.wb[l][((26 - t) * 16 + k) * kb + o] = h;
        }
        off += nw + co;
    }
}

// BF16 weight layouts from the FP32 master W[t][ci][co] of one layer:
//   forward  wf[t][n][k]  = W[t][k][n]          (k < kpad, n < 16; zero padded)
//   backward wb[t][n][k]  = W[26 - t][n][k]     (n = ci < 16, k = co < kpad)
__global__ void k_nn_pack(const float *__restrict__ W, int ci, int co, int kf, int ntf, uint16_t *__restrict__ wf,
                          int kb, int ntb, uint16_t *__restrict__ wb) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    int nf = ntf * 16 * kf;
    if (e < nf) {
        int t = e / (16 * kf), n = (e / kf) % 16, k = e % kf;
        float val = (t < 27 && n < co && k < ci) ? W[(t * ci + k) * co + n] : 0.f;
        wf[e] = to_bf16(val);
    }
    if (wb) {
        int nb = ntb * 16 * kb;
        if (e < nb) {
            int t = e / (16 * kb), n = (e / kb) % 16, k = e % kb;
            float val = (t < 27 && n < ci && k < co) ? W[((26 - t) * ci + n) * co + k] : 0.f;
            wb[e] = to_bf16(val);
        }
    }
}

int layer_off(int l) {
    int off = 0;
    for (int q = 0; q < l; q++) off += 27 * kNnChan[q] * kNnChan[q + 1] + kNnChan[q + 1];
    return off;
}

}  // namespace

// ---- host ----------------------------------------------------------------------
bo_status nn_pack(bo_nn *nn, hipStream_t s) {
    for (int l = 0; l < kNnLayers; l++) {
        int ci = kNnChan[l], co = kNnChan[l + 1];
        int kf = l == 0 ? 4 : 16, ntf = l == 0 ? 32 : 28;
        BO_TRY(nn->wf[l].alloc((size_t)ntf * 16 * kf));
        uint16_t *wb = nullptr;
        int kb = 16, ntb = 28;
        if (l > 0) {
            kb = l == kNnLayers - 1 ? 4 : 16;
            ntb = kb == 4 ? 32 : 28;
            BO_TRY(nn->wb[l].alloc((size_t)ntb * 16 * kb));
            wb = nn->wb[l].p;
        }
        int n = std::max(ntf * 16 * kf, ntb * 16 * kb);
        k_nn_pack<<<grid_for(n), kBlock, 0, s>>>(nn->w.p + layer_off(l), ci, co, kf, ntf, nn->wf[l].p, kb, ntb, wb);
    }
    BO_HIP(hipGetLastError());
    return BO_OK;
}

static bo_status nn_buffers(bo_nn *nn, const Vol &V) {
    size_t nv = (size_t)V.voxels();
    BO_TRY(nn->x1.alloc(4 * nv));
    BO_TRY(nn->a1.alloc(16 * nv));
    BO_TRY(nn->a2.alloc(16 * nv));
    BO_TRY(nn->a3.alloc(16 * nv));
    BO_TRY(nn->y.alloc(nv));
    nn->vol = V;
    return BO_OK;
}

// workgroups of a pass over nt tiles: a multiple of 8, at most what the chip
// holds at once (256 CUs, four workgroups each)
static unsigned conv_grid(long long nt, long long most = 1024) {
    return (unsigned)(std::min<long long>((nt + 7) / 8 * 8, most));
}

// forward pass of the network on x1 (already filled); the output lands in nn->y
// and, unless out is NULL, in out
static bo_status nn_forward_x1(bo_nn *nn, const Vol &V, float *out, hipStream_t s) {
    const long long nt = tiles_of(V);
    if (nt <= 0) return BO_OK;
    const float *w = nn->w.p;
    const unsigned nb = conv_grid(nt);
    k_nn_conv<4, MODE_ACT><<<nb, 256, 0, s>>>(V, (int)nt, nn->x1.p, nn->wf[0].p, w + layer_off(0) + 27 * 2 * 16,
                                              nullptr, nn->a1.p, nullptr, nullptr);
    k_nn_conv<16, MODE_ACT><<<nb, 256, 0, s>>>(V, (int)nt, nn->a1.p, nn->wf[1].p, w + layer_off(1) + 27 * 16 * 16,
                                               nullptr, nn->a2.p, nullptr, nullptr);
    k_nn_conv<16, MODE_ACT><<<nb, 256, 0, s>>>(V, (int)nt, nn->a2.p, nn->wf[2].p, w + layer_off(2) + 27 * 16 * 16,
                                               nullptr, nn->a3.p, nullptr, nullptr);
    k_nn_conv<16, MODE_OUT><<<nb, 256, 0, s>>>(V, (int)nt, nn->a3.p, nn->wf[3].p, w + layer_off(3) + 27 * 16,
                                               nullptr, nullptr, nn->y.p, out);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

// BF16 network input for CPR: channel 0 = r_p / s, channel 1 = standardised
// log-permeability (FP32, per cell)
template <typename T>
__global__ void k_nn_input_cpr(long long n, const T *__restrict__ rp, const double *__restrict__ s2,
                               const float *__restrict__ z, uint16_t *__restrict__ x) {
    long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    double s = sqrt(*s2);
    float r = (float)((double)rp[v] / (s > 0.0 ? s : 1.0));
    uint32_t h0 = to_bf16(r), h1 = to_bf16(z[v]);
    *(uint2 *)(x + 4 * v) = make_uint2(h0 | (h1 << 16), 0u);
}
template __global__ void k_nn_input_cpr<double>(long long, const double *, const double *, const float *, uint16_t *);
template __global__ void k_nn_input_cpr<float>(long long, const float *, const double *, const float *, uint16_t *);

bo_status nn_input_cpr(bo_nn *nn, const Grid &g, const void *rp, bool fp32, const double *s2, const float *z,
                       hipStream_t s) {
    Vol V;
    V.nb = 1; V.nz = g.nz; V.ny = g.ny; V.nx = g.nx;
    BO_TRY(nn_buffers(nn, V));
    nn->last_from_cpr = true;
    long long n = V.voxels();
    if (fp32) k_nn_input_cpr<float><<<grid_for(n), kBlock, 0, s>>>(n, (const float *)rp, s2, z, nn->x1.p);
    else k_nn_input_cpr<double><<<grid_for(n), kBlock, 0, s>>>(n, (const double *)rp, s2, z, nn->x1.p);
    BO_HIP(hipGetLastError());
    return nn_forward_x1(nn, V, nullptr, s);
}

}  // namespace bo

using namespace bo;

extern "C" bo_status bo_nn_create(bo_nn **out) {
    if (!out) return fail(BO_ERR_INVALID_ARG, "bo_nn_create: out is NULL");
    *out = nullptr;
    bo_nn *nn = new (std::nothrow) bo_nn();
    if (!nn) return fail(BO_ERR_ALLOC, "bo_nn_create: out of host memory");
    bo_status st = BO_OK;
    if ((st = nn->w.alloc(kNnParams)) || (st = nn->g.alloc(kNnParams)) || (st = nn->m.alloc(kNnParams)) ||
        (st = nn->v.alloc(kNnParams)) || (st = nn->lpart.alloc(1)) || (st = nn->loss.alloc(1))) {
        delete nn;
        return st;
    }
    if (hipMemset(nn->w.p, 0, sizeof(float) * kNnParams) != hipSuccess ||
        hipMemset(nn->g.p, 0, sizeof(float) * kNnParams) != hipSuccess ||
        hipMemset(nn->m.p, 0, sizeof(float) * kNnParams) != hipSuccess ||
        hipMemset(nn->v.p, 0, sizeof(float) * kNnParams) != hipSuccess) {
        delete nn;
        return fail(BO_ERR_HIP, "bo_nn_create: hipMemset failed");
    }
    if ((st = nn_pack(nn, nullptr)) != BO_OK || hipDeviceSynchronize() != hipSuccess) {
        delete nn;
        return st != BO_OK ? st : fail(BO_ERR_HIP, "bo_nn_create: packing the weights failed");
    }
    *out = nn;
    return BO_OK;
}

extern "C" void bo_nn_destroy(bo_nn *nn) {
    if (!nn) return;
    (void)hipDeviceSynchronize();
    delete nn;
}

extern "C" int32_t bo_nn_num_params(void) { return kNnParams; }

extern "C" bo_status bo_nn_set_params(bo_nn *nn, const float *params, void *stream) {
    if (!nn || !params) return fail(BO_ERR_INVALID_ARG, "bo_nn_set_params: NULL argument");
    hipStream_t s = (hipStream_t)stream;
    BO_HIP(hipMemcpyAsync(nn->w.p, params, sizeof(float) * kNnParams, hipMemcpyHostToDevice, s));
    BO_HIP(hipMemsetAsync(nn->m.p, 0, sizeof(float) * kNnParams, s));
    BO_HIP(hipMemsetAsync(nn->v.p, 0, sizeof(float) * kNnParams, s));
    nn->step = 0;
    BO_TRY(nn_pack(nn, s));
    BO_HIP(hipStreamSynchronize(s));
    return BO_OK;
}

extern "C" bo_status bo_nn_get_params(bo_nn *nn, float *params, float *grads, void *stream) {
    if (!nn) return fail(BO_ERR_INVALID_ARG, "bo_nn_get_params: NULL handle");
    hipStream_t s = (hipStream_t)stream;
    // through pinned memory: both copies are asynchronous and share one wait
    constexpr size_t bytes = sizeof(float) * kNnParams;
    if (!nn->pin) {
        const hipError_t e = hipHostMalloc((void **)&nn->pin, 2 * bytes, hipHostMallocDefault);
        if (e != hipSuccess) {
            nn->pin = nullptr;
            return fail(BO_ERR_ALLOC, std::string("bo_nn_get_params: hipHostMalloc failed: ") + hipGetErrorString(e));
        }
    }
    if (params) BO_HIP(hipMemcpyAsync(nn->pin, nn->w.p, bytes, hipMemcpyDeviceToHost, s));
    if (grads) BO_HIP(hipMemcpyAsync(nn->pin + kNnParams, nn->g.p, bytes, hipMemcpyDeviceToHost, s));
    BO_HIP(hipStreamSynchronize(s));
    if (params) std::memcpy(params, nn->pin, bytes);
    if (grads) std::memcpy(grads, nn->pin + kNnParams, bytes);
    return BO_OK;
}

extern "C" bo_status bo_nn_forward(bo_nn *nn, const float *in, float *out, int32_t nb, int32_t nz, int32_t ny,
                                   int32_t nx, void *stream) {
    if (!nn || !in || !out) return fail(BO_ERR_INVALID_ARG, "bo_nn_forward: NULL argument");
    if (nb < 1 || nz < 1 || ny < 1 || nx < 1) return fail(BO_ERR_INVALID_ARG, "bo_nn_forward: empty volume");
    Vol V;
    V.nb = nb; V.nz = nz; V.ny = ny; V.nx = nx;
    if (tiles_of(V) >= (1LL << 31)) return fail(BO_ERR_INVALID_ARG, "bo_nn_forward: volume too large");
    hipStream_t s = (hipStream_t)stream;
    BO_TRY(nn_buffers(nn, V));
    nn->last_from_cpr = false;
    long long nv = V.voxels();
    k_nn_input<<<grid_for(nv), kBlock, 0, s>>>(nv, in, nn->x1.p);
    BO_HIP(hipGetLastError());
    return nn_forward_x1(nn, V, out, s);
}

namespace {
// gradients of every layer from the output gradient in nn->dz4; the loss in
// nn->loss is copied to *loss (may be NULL); synchronises the stream
bo_status nn_backprop(bo_nn *nn, const Vol &V, double *loss, hipStream_t s) {
    const long long nt = tiles_of(V);
    const unsigned nb = conv_grid(nt), wb = conv_grid(nt, kNnWgradBlocks);
    BO_TRY(nn->part.alloc((size_t)wb * kNnPartStride));
    float *pt = nn->part.p;
    const int n = (int)nt;
    // layer 4 (A3 -> y)
    k_nn_wgrad<16, 16, 4, 1><<<wb, 384, 0, s>>>(V, n, nn->a3.p, nn->dz4.p, pt + layer_off(3));
    k_nn_conv<4, MODE_GRAD><<<nb, 256, 0, s>>>(V, n, nn->dz4.p, nn->wb[3].p, nullptr, nn->a3.p, nn->dz.p, nullptr,
                                               nullptr);
    // layer 3 (A2 -> A3)
    k_nn_wgrad<16, 16, 16, 16><<<wb, 384, 0, s>>>(V, n, nn->a2.p, nn->dz.p, pt + layer_off(2));
    k_nn_conv<16, MODE_GRAD><<<nb, 256, 0, s>>>(V, n, nn->dz.p, nn->wb[2].p, nullptr, nn->a2.p, nn->dzb.p, nullptr,
                                                nullptr);
    // layer 2 (A1 -> A2)
    k_nn_wgrad<16, 16, 16, 16><<<wb, 384, 0, s>>>(V, n, nn->a1.p, nn->dzb.p, pt + layer_off(1));
    k_nn_conv<16, MODE_GRAD><<<nb, 256, 0, s>>>(V, n, nn->dzb.p, nn->wb[1].p, nullptr, nn->a1.p, nn->dz.p, nullptr,
                                                nullptr);
    // layer 1 (X1 -> A1)
    k_nn_wgrad<4, 2, 16, 16><<<wb, 384, 0, s>>>(V, n, nn->x1.p, nn->dz.p, pt + layer_off(0));
    k_nn_wgrad_reduce<<<grid_for(kNnParams, 64), 512, 0, s>>>((int)wb, pt, nn->g.p);
    BO_HIP(hipGetLastError());
    if (loss) {
        const HostRead rd{nn->loss.p, sizeof(double), loss};
        return host_reads(&rd, 1, s);
    }
    BO_HIP(hipStreamSynchronize(s));
    return BO_OK;
}

bo_status nn_backward_check(bo_nn *nn, const char *who) {
    long long nv = nn->vol.voxels();
    if (nv <= 0 || nn->last_from_cpr)
        return fail(BO_ERR_INVALID_ARG, std::string(who) + ": the last forward pass was not a bo_nn_forward call");
    BO_TRY(nn->dz4.alloc(4 * (size_t)nv));
    BO_TRY(nn->dz.alloc(16 * (size_t)nv));
    BO_TRY(nn->dzb.alloc(16 * (size_t)nv));
    BO_TRY(nn->lpart.alloc(grid_for(nv)));
    return BO_OK;
}
}  // namespace

extern "C" bo_status bo_nn_backward(bo_nn *nn, const float *target, double *loss, void *stream) {
    if (!nn || !target) return fail(BO_ERR_INVALID_ARG, "bo_nn_backward: NULL argument");
    BO_TRY(nn_backward_check(nn, "bo_nn_backward"));
    const Vol V = nn->vol;
    long long nv = V.voxels();
    hipStream_t s = (hipStream_t)stream;
    unsigned nlb = grid_for(nv);
    k_nn_loss<<<nlb, 256, 0, s>>>(nv, nn->y.p, target, (float)(2.0 / (double)nv), nn->dz4.p, nn->lpart.p);
    k_nn_loss_final<<<1, kBlock, 0, s>>>((int)nlb, nn->lpart.p, 1.0 / (double)nv, nn->loss.p);
    return nn_backprop(nn, V, loss, s);
}

extern "C" bo_status bo_nn_backward_weighted(bo_nn *nn, const float *coef, const float *target, double *loss,
                                             void *stream) {
    if (!nn || !coef || !target) return fail(BO_ERR_INVALID_ARG, "bo_nn_backward_weighted: NULL argument");
    BO_TRY(nn_backward_check(nn, "bo_nn_backward_weighted"));
    const Vol V = nn->vol;
    long long nv = V.voxels();
    long long interior = (long long)V.nb * std::max(V.nz - 2, 0) * std::max(V.ny - 2, 0) * std::max(V.nx - 2, 0);
    if (interior <= 0)
        return fail(BO_ERR_INVALID_ARG, "bo_nn_backward_weighted: the volume has no interior voxel (a side below 3)");
    hipStream_t s = (hipStream_t)stream;
    unsigned nlb = grid_for(nv);
    BO_TRY(nn->wres.alloc((size_t)nv));
    k_nn_wres<<<nlb, 256, 0, s>>>(V, coef, nn->y.p, target, nn->wres.p, nn->lpart.p);
    k_nn_loss_final<<<1, kBlock, 0, s>>>((int)nlb, nn->lpart.p, 1.0 / (double)interior, nn->loss.p);
    k_nn_wout<<<nlb, kBlock, 0, s>>>(V, coef, nn->wres.p, (float)(2.0 / (double)interior), nn->dz4.p);
    return nn_backprop(nn, V, loss, s);
}

extern "C" bo_status bo_nn_adam_step(bo_nn *nn, float lr, void *stream) {
    if (!nn) return fail(BO_ERR_INVALID_ARG, "bo_nn_adam_step: NULL handle");
    if (!(lr > 0.f)) return fail(BO_ERR_INVALID_ARG, "bo_nn_adam_step: lr must be positive");
    hipStream_t s = (hipStream_t)stream;
    nn->step++;
    const float b1 = 0.9f, b2 = 0.999f;
    float c1 = (float)(1.0 - std::pow(0.9, (double)nn->step));
    float c2 = (float)(1.0 - std::pow(0.999, (double)nn->step));
    PackedNet P;
    for (int l = 0; l < kNnLayers; l++) {
        P.wf[l] = nn->wf[l].p;
        P.wb[l] = nn->wb[l].p;
    }
    k_nn_adam<<<grid_for(kNnParams), kBlock, 0, s>>>(kNnParams, nn->w.p, nn->g.p, nn->m.p, nn->v.p, lr, b1, b2,
                                                     1e-8f, c1, c2, P);
    BO_HIP(hipGetLastError());
    return BO_OK;
}
