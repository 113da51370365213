// F stage of CPR (Section 3.2): the paper's restricted additive Schwarz with
// ILU(0) subdomain solves, mapped onto the GPU as non-overlapping subdomains
// of tile_x x tile_y grid columns (all nz layers), one wavefront per tile.
//
// On the 7-point stencil the grid graph has no triangles, so block ILU(0)
// only modifies the diagonal blocks: E_i = A_ii - sum_{k<i} A_ik E_k^{-1} A_ki
// over the lower neighbours k inside the tile (natural order: -z, -y, -x).
// The FP64 solve takes the unit-lower factors L_ik = A_ik E_k^{-1}:
// y_i = r_i - sum_{k<i} L_ik y_k, then x_i = E_i^{-1}(y_i - sum_{j>i} A_ij x_j)
// (27 factor values per cell forward, 36 backward).  The FP32 / BF16 forms
// keep the blocks of A: w_i = E_i^{-1}(r_i - sum_{k<i} A_ik w_k), then
// x_i = w_i - E_i^{-1} sum_{j>i} A_ij x_j.
//
// Schedule: lane t = a + tile_x*b of the tile owns grid column (i0+a, j0+b)
// and at step s handles layer k = s - a - b, so its -x, -y and -z neighbours
// were handled one step earlier by lanes t-1, t-tile_x and t itself.  The
// factors are stored in the same (tile, step, lane) order, packed in pairs, so
// each step reads its doubles with contiguous 1 KB loads (14 or 18 of them),
// several steps ahead (see the sweeps below).
// Block Jacobi (x_i = A_ii^{-1} r_i) is the alternative F stage.
//
// Mixed form: the factors (E^{-1} and the blocks of A) are computed in FP64
// and stored rounded to FP32 (9 float4 per slot and sweep) or to BF16 (9 uint2
// per slot and sweep, round to nearest even from the FP32 value); the sweeps
// run in FP32 on FP32 vectors.
#include <type_traits>
#include "bo_cpr.hpp"

namespace bo {
namespace {

struct TileGeom {
    int nx, ny, nz, tx, ty, ntx, nty, ns;
    __host__ __device__ long long slots() const { return (long long)ntx * nty * ns * 64; }
};

// The factors of one slot for one sweep are 36 doubles: E^{-1} and the three
// lower blocks (-z, -y, -x) for the forward sweep, E^{-1} and the three upper
// blocks (+z, +x, +y) for the backward sweep.  They are packed as 18 double2
// per slot in (tile, step, pair, lane) order, so one wavefront load of a
// pair reads 1 KB contiguously and a step needs 18 load instructions.  In the
// FP64 form the forward slot holds the unit-lower factors in place of the
// lower blocks and its sweep reads pairs 4..17 only (values 8..35).
constexpr int kPairs = 18;
__device__ __forceinline__ size_t pk_index(int tile, int ns, int s, int pair, int lane) {
    return (((size_t)tile * ns + s) * kPairs + pair) * 64 + lane;
}

enum { ST_F64 = 0, ST_F32 = 1, ST_BF16 = 2 };
constexpr int kQuads = 9;  // 36 values as 9 groups of four (FP32 / BF16 forms)
__device__ __forceinline__ size_t pq_index(int tile, int ns, int s, int quad, int lane) {
    return (((size_t)tile * ns + s) * kQuads + quad) * 64 + lane;
}

// FP32 -> BF16, round to nearest even (inputs are finite)
__device__ __forceinline__ uint32_t bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ float bf16_value(uint32_t h) { return __uint_as_float(h << 16); }

// store one slot's 36 FP64 values in the chosen format
template <int St>
__device__ __forceinline__ void store_pack(void *F, int tile, int ns, int s, int t, const double *v) {
    if constexpr (St == ST_F64) {
        double2 *D = (double2 *)F;
        for (int p2 = 0; p2 < kPairs; p2++) D[pk_index(tile, ns, s, p2, t)] = make_double2(v[2 * p2], v[2 * p2 + 1]);
    } else if constexpr (St == ST_F32) {
        float4 *D = (float4 *)F;
        for (int qd = 0; qd < kQuads; qd++)
            D[pq_index(tile, ns, s, qd, t)] = make_float4((float)v[4 * qd], (float)v[4 * qd + 1],
                                                          (float)v[4 * qd + 2], (float)v[4 * qd + 3]);
    } else {
        uint2 *D = (uint2 *)F;
        for (int qd = 0; qd < kQuads; qd++) {
            uint32_t h0 = bf16_bits((float)v[4 * qd]), h1 = bf16_bits((float)v[4 * qd + 1]);
            uint32_t h2 = bf16_bits((float)v[4 * qd + 2]), h3 = bf16_bits((float)v[4 * qd + 3]);
            D[pq_index(tile, ns, s, qd, t)] = make_uint2(h0 | (h1 << 16), h2 | (h3 << 16));
        }
    }
}

__device__ __forceinline__ void load_blk(const double *__restrict__ A, int slot, size_t N, int g, double *o) {
    const double *p = A + (size_t)slot * 9 * N + g;
#pragma unroll
    for (int z = 0; z < 9; z++) o[z] = p[(size_t)z * N];
}

template <typename T>
__device__ __forceinline__ void mv3(const T *A, const T *x, T *y) {
    y[0] = A[0] * x[0] + A[1] * x[1] + A[2] * x[2];
    y[1] = A[3] * x[0] + A[4] * x[1] + A[5] * x[2];
    y[2] = A[6] * x[0] + A[7] * x[1] + A[8] * x[2];
}

template <int K>
__device__ __forceinline__ void shfl_arr(const double *src, double *dst, int lane) {
#pragma unroll
    for (int z = 0; z < K; z++) dst[z] = __shfl(src[z], lane, 64);
}

// Factorisation in two passes, in FP64 for every storage format.  Pack: the
// blocks of every slot (tile, step, lane) into the FP64 packed layout (forward
// slot: [A_ii | Az Ay Ax] with the lower blocks -z, -y, -x; backward slot:
// [- | Uz Ux Uy] with the upper blocks +z, +x, +y; zero where the neighbour
// lies outside the tile or grid), and the slot of each cell.  Chain: one
// wavefront per tile walks the steps; lane t = a + tile_x*b at step s handles
// layer k = s - a - b and forms E_i = A_ii - sum over -z, -y, -x of
// (A_ik E_k^{-1}) U_ki from the values its neighbours held one step earlier
// (shuffled), reading each step's blocks from the packed layout (1 KB per load
// instruction), and E_i^{-1} by Gauss-Jordan with partial pivoting.
//
// The pack is bound by the memory it reads and writes.  The lanes of a step
// lie in as many layers as the tile is wide, so a thread gathering its own
// slot reads 64 separate sectors per load, and the cells beside them come in
// later steps: eight times the matrix through the L2.  A workgroup takes
// kPackSteps steps of a tile instead (as many more as a wavefront holds tiles) and
// reads runs of that many cells of a tile's rows at one layer, 18 planes at a time
// (two blocks), into LDS at their slots: in pass f lane (a, b) takes step (f + a)
// mod steps, so that all lanes work in every pass whatever the tile's width.
// 2 M cells, a thread per slot and now: tiles of 8x8 978 and 647 us (2.1 GB), of
// 16x4 1223 and 608, of 4x4 1241 and 607, of 3x2 1330 and 702, of 64x1 758 and 562
// us; with passes by layer, where lanes without a step in the chunk idle, 8x8 628,
// 3x2 1705, 64x1 976 us.  Chunks of 4 steps 684 us, workgroups dealt to the
// XCDs in turn instead of in ranges 702 us (8x8).
constexpr int kPackSteps = 8;
__host__ __device__ inline int pack_steps(const TileGeom &T) { return kPackSteps * (64 / (T.tx * T.ty)); }
__global__ void __launch_bounds__(kBlock) k_ilu_pack(TileGeom T, const double *__restrict__ A,
                                                     double2 *__restrict__ Ff, double2 *__restrict__ Fb,
                                                     int32_t *__restrict__ slot_of) {
    __shared__ double buf[18][kPackSteps * 64];
    const int cols = T.tx * T.ty, sets = 64 / cols, steps = pack_steps(T);
    const int chunks = (T.ns + steps - 1) / steps;
    const int wg = xcd_block(blockIdx.x, gridDim.x);
    const int tile = wg / chunks, s0 = (wg % chunks) * steps;
    const int ti = tile % T.ntx, tj = tile / T.ntx;
    // a wavefront takes as many layers (or steps) at a time as it holds a tile's columns
    const int t = threadIdx.x % 64 % cols, set = threadIdx.x % 64 / cols, first = threadIdx.x / 64 * sets + set;
    const int a = t % T.tx, b = t / T.tx;
    const int i = ti * T.tx + a, j = tj * T.ty + b;
    const bool column = set < sets && i < T.nx && j < T.ny;
    const bool has_mx = a > 0, has_my = b > 0;
    const bool has_px = a + 1 < T.tx && i + 1 < T.nx, has_py = b + 1 < T.ty && j + 1 < T.ny;
    const size_t N = (size_t)T.nx * T.ny * T.nz;
    // blocks 2h and 2h + 1 of [A_ii Az Ay Ax - Uz Ux Uy]
#pragma unroll 1
    for (int h = 0; h < 4; h++) {
        const int sl0 = h == 0 ? S_D : h == 1 ? S_MY : h == 2 ? -1 : S_PX;
        const int sl1 = h == 0 ? S_MZ : h == 1 ? S_MX : h == 2 ? S_PZ : S_PY;
        // pass f: step s0 + u of each lane, u = (f + a) mod steps, so that runs of
        // `steps` lanes of a row read one layer
        for (int f = first; f < steps; f += kBlock / 64 * sets) {
            const int u = (f + a) % steps, k = s0 + u - a - b;
            if (!(column && k >= 0 && k < T.nz)) continue;
            const bool h0 = h == 0 ? true : h == 1 ? has_my : h == 2 ? false : has_px;
            const bool h1 = h == 0 ? k > 0 : h == 1 ? has_mx : h == 2 ? k + 1 < T.nz : has_py;
            const int g = i + T.nx * (j + T.ny * k);
            double x[18];
            if (h0) load_blk(A, sl0, N, g, x);
            else
                for (int z = 0; z < 9; z++) x[z] = 0.0;
            if (h1) load_blk(A, sl1, N, g, x + 9);
            else
                for (int z = 9; z < 18; z++) x[z] = 0.0;
#pragma unroll
            for (int z = 0; z < 18; z++) buf[z][u * cols + t] = x[z];
        }
        __syncthreads();
        for (int u = first; u < steps; u += kBlock / 64 * sets) {
            const int s = s0 + u, k = s - a - b;
            if (!(column && s < T.ns && k >= 0 && k < T.nz)) continue;  // idle slot
            double2 *const F = h < 2 ? Ff : Fb;
#pragma unroll
            for (int p = 0; p < 9; p++) {
                if (h == 2 && p < 4) continue;  // values 0..7 of the backward slot: the chain's
                F[pk_index(tile, T.ns, s, (h & 1) * 9 + p, t)] =
                    make_double2(buf[2 * p][u * cols + t], buf[2 * p + 1][u * cols + t]);
            }
            if (h == 0) slot_of[i + T.nx * (j + T.ny * k)] = (int32_t)(((long long)tile * T.ns + s) * 64 + t);
        }
        __syncthreads();
    }
}

// The same pack straight from a BSR matrix whose first N block rows are the
// grid's cells, each row's stencil blocks first in ascending column order
// (the extended grid form; later columns, matrix cells or wells, follow):
// the thread reads its cell's row (contiguous blocks) instead of 63 slot
// planes.  A stencil neighbour missing from the row raises *bad.
__global__ void __launch_bounds__(kBlock) k_ilu_pack_bsr(TileGeom T, const int32_t *__restrict__ rp,
                                                         const int32_t *__restrict__ ci,
                                                         const double *__restrict__ v, double2 *__restrict__ Ff,
                                                         double2 *__restrict__ Fb, int32_t *__restrict__ slot_of,
                                                         int32_t *__restrict__ bad) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= T.slots()) return;
    const int t = (int)(q % 64);
    const long long ts = q / 64;
    const int s = (int)(ts % T.ns), tile = (int)(ts / T.ns);
    const int a = t % T.tx, b = t / T.tx;
    const int ti = tile % T.ntx, tj = tile / T.ntx;
    const int i = ti * T.tx + a, j = tj * T.ty + b, k = s - a - b;
    if (!(t < T.tx * T.ty && i < T.nx && j < T.ny && k >= 0 && k < T.nz)) return;  // idle slot
    const int g = i + T.nx * (j + T.ny * k);
    // grid neighbours present (slot order) and the blocks the tile keeps
    const unsigned have = (k > 0 ? 1u << S_MZ : 0u) | (j > 0 ? 1u << S_MY : 0u) | (i > 0 ? 1u << S_MX : 0u) |
                          (1u << S_D) | (i + 1 < T.nx ? 1u << S_PX : 0u) | (j + 1 < T.ny ? 1u << S_PY : 0u) |
                          (k + 1 < T.nz ? 1u << S_PZ : 0u);
    const unsigned keep = (k > 0 ? 1u << S_MZ : 0u) | (b > 0 ? 1u << S_MY : 0u) | (a > 0 ? 1u << S_MX : 0u) |
                          (1u << S_D) | (a + 1 < T.tx && i + 1 < T.nx ? 1u << S_PX : 0u) |
                          (b + 1 < T.ty && j + 1 < T.ny ? 1u << S_PY : 0u) | (k + 1 < T.nz ? 1u << S_PZ : 0u);
    const int e0 = rp[g], e1 = rp[g + 1];
    const int nxy = T.nx * T.ny;
    const int nb[NSLOT] = {g - nxy, g - T.nx, g - 1, g, g + 1, g + T.nx, g + nxy};
    int pos[NSLOT];
    int c[NSLOT];
#pragma unroll
    for (int sl = 0; sl < NSLOT; sl++) {
        pos[sl] = e0 + __popc(have & ((1u << sl) - 1u));
        c[sl] = (have >> sl) & 1u ? ci[min(pos[sl], e1 - 1)] : -1;
    }
    bool ok = true;
#pragma unroll
    for (int sl = 0; sl < NSLOT; sl++)
        if ((have >> sl) & 1u) ok = ok && pos[sl] < e1 && c[sl] == nb[sl];
    if (!ok) {
        *bad = 1;
        return;
    }
    // fw = [A_ii | -z | -y | -x], bw[9..35] = [+z | +x | +y]; zero blocks outside the tile
    const int fsl[4] = {S_D, S_MZ, S_MY, S_MX}, bsl[3] = {S_PZ, S_PX, S_PY};
    double fw[36], bw[27];
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const bool k_ = (keep >> fsl[u]) & 1u;
        const double *src = v + 9 * (size_t)(k_ ? pos[fsl[u]] : e0);
#pragma unroll
        for (int z = 0; z < 9; z++) fw[9 * u + z] = k_ ? src[z] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 3; u++) {
        const bool k_ = (keep >> bsl[u]) & 1u;
        const double *src = v + 9 * (size_t)(k_ ? pos[bsl[u]] : e0);
#pragma unroll
        for (int z = 0; z < 9; z++) bw[9 * u + z] = k_ ? src[z] : 0.0;
    }
#pragma unroll
    for (int p2 = 0; p2 < kPairs; p2++) {
        Ff[pk_index(tile, T.ns, s, p2, t)] = make_double2(fw[2 * p2], fw[2 * p2 + 1]);
        if (p2 >= 5) Fb[pk_index(tile, T.ns, s, p2, t)] = make_double2(bw[2 * p2 - 9], bw[2 * p2 - 8]);
    }
    // pair 4 of the backward slot: (E^{-1}[8], +z[0]); the chain writes E^{-1}
    Fb[pk_index(tile, T.ns, s, 4, t)] = make_double2(0.0, bw[0]);
    slot_of[g] = (int32_t)q;
}

// one slot of the FP32 / BF16 forms: values 0..8 from e, 9..35 from r (the
// three blocks of A), rounded to nearest
template <int St>
__device__ __forceinline__ void store_mixed(void *F, int tile, int ns, int s, int t, const double *e,
                                            const double *r) {
#pragma unroll
    for (int qd = 0; qd < kQuads; qd++) {
        float f[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int z = 4 * qd + u;
            f[u] = (float)(z < 9 ? e[z] : r[z - 9]);
        }
        if constexpr (St == ST_F32) {
            ((float4 *)F)[pq_index(tile, ns, s, qd, t)] = make_float4(f[0], f[1], f[2], f[3]);
        } else {
            ((uint2 *)F)[pq_index(tile, ns, s, qd, t)] =
                make_uint2(bf16_bits(f[0]) | (bf16_bits(f[1]) << 16), bf16_bits(f[2]) | (bf16_bits(f[3]) << 16));
        }
    }
}

// FP64 form: E^{-1} and the unit-lower factors over the packed input (Ff,
// Fb).  FP32 / BF16 forms: the packed input is left as it is and each slot
// is stored rounded into Of ([E^{-1} | Az Ay Ax]) and Ob ([E^{-1} | Uz Ux
// Uy]), the blocks of A as the sweeps of those forms take them.
template <int St>
__global__ void __launch_bounds__(64) k_ilu_chain(TileGeom T, double2 *__restrict__ Ff, double2 *__restrict__ Fb,
                                                  int32_t *__restrict__ bad, double *__restrict__ einv_nat,
                                                  void *__restrict__ Of, void *__restrict__ Ob) {
    int t = threadIdx.x;
    int a = t % T.tx, b = t / T.tx;
    int tile = blockIdx.x;
    int ti = tile % T.ntx, tj = tile / T.ntx;
    int i = ti * T.tx + a, j = tj * T.ty + b;
    bool active = t < T.tx * T.ty && i < T.nx && j < T.ny;
    bool has_mx = a > 0, has_my = b > 0;
    size_t N = (size_t)T.nx * T.ny * T.nz;
    double Ep[9], Uxp[9], Uyp[9], Uzp[9];  // this lane's values from the previous step
    for (int z = 0; z < 9; z++) Ep[z] = Uxp[z] = Uyp[z] = Uzp[z] = 0.0;
    // a step's 63 values, loaded one step ahead into a ring of two buffers
    // (the loop is unrolled by two so that no buffer is copied: a copy of
    // registers with loads in flight makes the compiler wait for all of them)
    struct Slot {
        double fw[36], uw[27];
    };
    auto fetch = [&](int s, Slot &S) {
        const int sc = min(s, T.ns - 1);
        const int k = sc - a - b;
        // every lane loads (idle lanes read lane 0's slot) so that no load
        // is skipped on some paths
        const int tl = active && k >= 0 && k < T.nz ? t : 0;
#pragma unroll
        for (int p2 = 0; p2 < kPairs; p2++) {
            double2 d = Ff[pk_index(tile, T.ns, sc, p2, tl)];
            S.fw[2 * p2] = d.x;
            S.fw[2 * p2 + 1] = d.y;
        }
        double2 d = Fb[pk_index(tile, T.ns, sc, 4, tl)];
        S.uw[0] = d.y;
#pragma unroll
        for (int p2 = 5; p2 < kPairs; p2++) {
            double2 e = Fb[pk_index(tile, T.ns, sc, p2, tl)];
            S.uw[2 * p2 - 9] = e.x;
            S.uw[2 * p2 - 8] = e.y;
        }
    };
    auto step = [&](int s, const Slot &S) {
        double Ex[9], Ey[9], Ux[9], Uy[9];
        shfl_arr<9>(Ep, Ex, has_mx ? t - 1 : t);
        shfl_arr<9>(Uxp, Ux, has_mx ? t - 1 : t);
        shfl_arr<9>(Ep, Ey, has_my ? t - T.tx : t);
        shfl_arr<9>(Uyp, Uy, has_my ? t - T.tx : t);
        int k = s - a - b;
        const bool act = active && k >= 0 && k < T.nz;
        const double *fw = S.fw, *uw = S.uw;
        if (act) {
            // lw: E^{-1}[8] and the unit-lower factors L_ik = A_ik E_k^{-1}
            // (-z, -y, -x) as values 8..35 of the forward slot
            double E[9], lw[28], tmp[9];
            for (int z = 0; z < 28; z++) lw[z] = 0.0;
            for (int z = 0; z < 9; z++) E[z] = fw[z];
            // -z, -y, -x in ascending order (zero blocks where missing)
            if (k > 0) {
                mul3(fw + 9, Ep, lw + 1); mul3(lw + 1, Uzp, tmp);
                for (int z = 0; z < 9; z++) E[z] = E[z] - tmp[z];
            }
            if (has_my) {
                mul3(fw + 18, Ey, lw + 10); mul3(lw + 10, Uy, tmp);
                for (int z = 0; z < 9; z++) E[z] = E[z] - tmp[z];
            }
            if (has_mx) {
                mul3(fw + 27, Ex, lw + 19); mul3(lw + 19, Ux, tmp);
                for (int z = 0; z < 9; z++) E[z] = E[z] - tmp[z];
            }
            double Ei[9];
            if (!inv3_gj(E, Ei)) {
                *bad = 1;
                for (int z = 0; z < 9; z++) Ei[z] = 0.0;
            }
            for (int z = 0; z < 9; z++) Ep[z] = Ei[z];
            if (einv_nat) {
                const int g = i + T.nx * (j + T.ny * k);
                for (int z = 0; z < 9; z++) einv_nat[(size_t)z * N + g] = Ei[z];
            }
            if constexpr (St != ST_F64) {
                store_mixed<St>(Of, tile, T.ns, s, t, Ei, fw + 9);
                store_mixed<St>(Ob, tile, T.ns, s, t, Ei, uw);
                for (int z = 0; z < 9; z++) { Uzp[z] = uw[z]; Uxp[z] = uw[9 + z]; Uyp[z] = uw[18 + z]; }
                return;
            }
            // E^{-1} into values 0..8 of the backward slot, the lower factors
            // over the forward slot's blocks of A (its values 0..7, A_ii, are
            // not read again)
#pragma unroll
            for (int p2 = 0; p2 < 4; p2++)
                Fb[pk_index(tile, T.ns, s, p2, t)] = make_double2(Ei[2 * p2], Ei[2 * p2 + 1]);
            ((double *)&Fb[pk_index(tile, T.ns, s, 4, t)])[0] = Ei[8];
            lw[0] = Ei[8];
#pragma unroll
            for (int p2 = 4; p2 < kPairs; p2++)
                Ff[pk_index(tile, T.ns, s, p2, t)] = make_double2(lw[2 * p2 - 8], lw[2 * p2 - 7]);
            // this cell's upper blocks for the next step's neighbours
            for (int z = 0; z < 9; z++) { Uzp[z] = uw[z]; Uxp[z] = uw[9 + z]; Uyp[z] = uw[18 + z]; }
        }
    };
    Slot R0, R1;
    fetch(0, R0);
    int s0 = 0;
    for (; s0 + 2 <= T.ns; s0 += 2) {
        fetch(s0 + 1, R1);
        step(s0, R0);
        fetch(s0 + 2, R0);
        step(s0 + 1, R1);
    }
    if (s0 < T.ns) step(s0, R0);
}

// One slot's factors as loaded, for one sweep: FP64 forward 14 pairs (4..17:
// a pad and the unit-lower factors -z, -y, -x), FP64 backward 18 pairs (E^-1,
// +z, +x, +y), FP32 / BF16 9 quads (E^-1 and three blocks).
template <int St, bool FWD>
struct Factors {
    typedef typename std::conditional<St == ST_F64, double2,
                                      typename std::conditional<St == ST_F32, float4, uint2>::type>::type Raw;
    static constexpr int kFirst = St == ST_F64 && FWD ? 4 : 0;
    static constexpr int kCount = St == ST_F64 ? kPairs - kFirst : kQuads;
    static constexpr int kStride = St == ST_F64 ? kPairs : kQuads;
    Raw raw[kCount];
    template <bool NT>
    __device__ __forceinline__ void load(const Raw *__restrict__ p) {
        typedef uint32_t V __attribute__((ext_vector_type(sizeof(Raw) / 4)));
#pragma unroll
        for (int i = 0; i < kCount; i++) {
            if constexpr (NT)
                raw[i] = __builtin_bit_cast(Raw, __builtin_nontemporal_load((const V *)(p + (kFirst + i) * 64)));
            else
                raw[i] = p[(kFirst + i) * 64];
        }
    }
    // values 9 q .. 9 q + 8 of the slot's 36 (q = 1..3 in the FP64 forward form)
    template <typename T>
    __device__ __forceinline__ void block(int q, T *o) const {
#pragma unroll
        for (int z = 0; z < 9; z++) {
            const int v = 9 * q + z;
            if constexpr (St == ST_F64) {
                const int w = v - 2 * kFirst;
                o[z] = w % 2 ? raw[w / 2].y : raw[w / 2].x;
            } else if constexpr (St == ST_F32) {
                const float4 f = raw[v / 4];
                o[z] = v % 4 == 0 ? f.x : v % 4 == 1 ? f.y : v % 4 == 2 ? f.z : f.w;
            } else {
                const uint32_t h = v % 4 < 2 ? raw[v / 4].x : raw[v / 4].y;
                o[z] = bf16_value(v % 2 ? h >> 16 : h & 0xFFFFu);
            }
        }
    }
};

// The sweeps: one wavefront per tile, no barrier.  Lane t = a + tile_x*b owns
// grid column (i0+a, j0+b) and at step s handles layer k = s - a - b; the
// neighbours' values of the previous step come by lane shuffles.  The loads of
// AH steps are in flight: a ring of register buffers, the step loop unrolled by
// its length, so a buffer is refilled in place once its step is done and no
// register with a load in flight is ever copied (a copy would wait for it).
// Every load and store is issued on every path (idle slots read another lane's
// data of the step, stores that have nothing to do repeat a value): the hardware
// returns vector memory operations in order and the compiler counts them
// statically, so one that some paths skip makes later waits take in the next
// steps' loads too.  (With conditional output stores and two wavefronts
// joined by two barriers a step took one memory latency whatever the ring's
// length: 1.17 us backward and 0.57 us forward on one tile, 0.46 us so; both
// sweeps of a 104x104x31 grid 76 and now 46 us, of a 100x100x50 grid 112 and 80
// us, where 169 tiles on 256 CUs reach 4 TB/s.)
// Idle slots read the data of a lane that has a cell, which is loaded anyway: lane
// 0's lines, where lane 0 is idle too, are a fifth of a one-layer grid's traffic
// (both sweeps of 1000x1000x1 in FP64 1045 and 950 us, in BF16 384 and 346 us).
// Finding that lane costs the mixed forms with few tiles, bound by the chain, more
// than the lines do (100x100x50 in BF16 55.8 us, 57.1 so).
struct SweepLane {
    int t, a, b, ab;  // ab: first step of the column, out of reach for a lane without one
    size_t c0;        // the column's cell in layer 0
    __device__ SweepLane(const TileGeom &G, int tile, int lane) : t(lane) {
        a = lane % G.tx;
        b = lane / G.tx;
        const int i = (tile % G.ntx) * G.tx + a, j = (tile / G.ntx) * G.ty + b;
        const bool col_ok = lane < G.tx * G.ty && i < G.nx && j < G.ny;
        ab = col_ok ? a + b : 1 << 30;
        c0 = (size_t)i + (size_t)G.nx * j;
    }
    __device__ __forceinline__ bool active(const TileGeom &G, int s) const {
        return (unsigned)(s - ab) < (unsigned)G.nz;
    }
    // the lane whose slot of step s this lane loads: its own, an idle one the
    // first lane's that has a cell (SHARE) or lane 0's
    template <bool SHARE>
    __device__ __forceinline__ int load_lane(const TileGeom &G, int s) const {
        const bool act = active(G, s);
        if constexpr (!SHARE) return act ? t : 0;
        const uint64_t m = __ballot(act);
        const int first = m ? __ffsll((unsigned long long)m) - 1 : 0;
        return act ? t : first;
    }
    // the grid cell of a slot (cell 0 for an idle one)
    __device__ __forceinline__ size_t cell(const TileGeom &G, int s) const {
        return active(G, s) ? c0 + (size_t)(s - ab) * ((size_t)G.nx * G.ny) : 0;
    }
};

// forward sweep: FP64: y = r - sum_lower L y_lower with the unit-lower
// factors L_ik = A_ik E_k^{-1}; FP32 / BF16: w = E^{-1}(r - sum_lower A w_lower)
// (w = E^{-1} y).  r (FP64) in natural order, read at the slot's cell and
// rounded to T; the result in (tile, step, lane) order
template <int St, typename T, int AH, bool NT>
__global__ void __launch_bounds__(64) k_ilu_forward(TileGeom G, const void *__restrict__ F,
                                                    const double *__restrict__ r, T *__restrict__ wq) {
    typedef Factors<St, true> Fac;
    const int tile = blockIdx.x, ns = G.ns;
    const SweepLane L(G, tile, threadIdx.x);
    const int t = L.t;
    const size_t S = (size_t)G.slots();
    const typename Fac::Raw *Ft = (const typename Fac::Raw *)F + (size_t)tile * ns * Fac::kStride * 64;
    T *wt = wq + (size_t)tile * ns * 64 + t;
    const int lx = L.a > 0 ? t - 1 : t, ly = L.b > 0 ? t - G.tx : t;
    struct Slot {
        Fac f;
        double r[3];
    } ring[AH];
    auto fetch = [&](int s, Slot &Q) {
        const int sc = min(s, ns - 1);
        Q.f.template load<NT>(Ft + (size_t)sc * Fac::kStride * 64 + L.template load_lane<AH == 2>(G, sc));
        const double *rg = r + 3 * L.cell(G, sc);
        Q.r[0] = rg[0]; Q.r[1] = rg[1]; Q.r[2] = rg[2];
    };
    T wp[3] = {0, 0, 0};
    auto step = [&](int s, const Slot &Q) {
        T wx[3], wy[3];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            wx[c] = __shfl(wp[c], lx, 64);
            wy[c] = __shfl(wp[c], ly, 64);
        }
        // zero blocks stand for missing neighbours
        T A[9], y[3], v[3] = {(T)Q.r[0], (T)Q.r[1], (T)Q.r[2]};
        Q.f.block(1, A);
        mv3(A, wp, y); v[0] = v[0] - y[0]; v[1] = v[1] - y[1]; v[2] = v[2] - y[2];
        Q.f.block(2, A);
        mv3(A, wy, y); v[0] = v[0] - y[0]; v[1] = v[1] - y[1]; v[2] = v[2] - y[2];
        Q.f.block(3, A);
        mv3(A, wx, y); v[0] = v[0] - y[0]; v[1] = v[1] - y[1]; v[2] = v[2] - y[2];
        if constexpr (St != ST_F64) {
            Q.f.block(0, A);
            mv3(A, v, y);
            v[0] = y[0]; v[1] = y[1]; v[2] = y[2];
        }
        const bool act = L.active(G, s);
        T *w = wt + (size_t)s * 64;  // idle slots store 0
#pragma unroll
        for (int c = 0; c < 3; c++) {
            wp[c] = act ? v[c] : (T)0;
            w[c * S] = wp[c];
        }
    };
    ring_steps<AH>(ns, ring, step, fetch);
}

// backward sweep: FP64: x_i = E_i^{-1}(y_i - sum_{upper} A_ij x_j); FP32 /
// BF16: x_i = w_i - E_i^{-1} sum_{upper} A_ij x_j; written in natural order as
// out = x + (dp, 0, 0) in FP64 (dp may be NULL), or with ZIN added to zin: out
// = zin + (x + (dp, 0, 0)) (zin may be out itself: each value is read and
// written by one wavefront, the read AH steps before).
// Output staging: lane (a, b) finishes layer k at step k + a + b, so the layers
// in flight at step s are s .. s + D - 1 (D = tile_x + tile_y - 1) and layer s
// is complete once step s is.  Each result goes into the layer's LDS slot (k
// mod D, 64 x 3 doubles); step s writes layer s + 1 to HBM as tile_y rows of 3
// tile_x contiguous doubles, three values per lane (lanes beyond the tile's or
// the grid's columns repeat the tile's first value; up to 2 AH - 1 steps before
// the first finished layer write the last layer's places, in the ZIN form with
// the values they hold).  Without staging (STAGE false, where D layers do not fit) every lane
// writes its 24 bytes at its cell, and the partial lines cost HBM writes of more than twice the output's size.
template <int St, typename T, typename TD, int AH, bool NT, bool ZIN, bool STAGE>
__global__ void __launch_bounds__(64) k_ilu_backward(TileGeom G, const void *__restrict__ F, T *__restrict__ wq,
                                                     const TD *__restrict__ dp, double *out, int D,
                                                     const double *zin) {
    extern __shared__ double obuf[];  // D slots of [lane][3]
    typedef Factors<St, false> Fac;
    const int tile = blockIdx.x, ns = G.ns, e = G.ns - 1;
    const SweepLane L(G, tile, threadIdx.x);
    const int t = L.t;
    const size_t S = (size_t)G.slots(), nxy3 = 3 * (size_t)G.nx * G.ny;
    const typename Fac::Raw *Ft = (const typename Fac::Raw *)F + (size_t)tile * ns * Fac::kStride * 64;
    T *wt = wq + (size_t)tile * ns * 64;
    const int px = L.a + 1 < G.tx && t + 1 < 64 ? t + 1 : t;
    const int py = L.b + 1 < G.ty && t + G.tx < 64 ? t + G.tx : t;
    // the three values of a finished layer this lane writes: place in the LDS
    // slot and in the layer
    int lo[3];
    size_t go[3];
    if constexpr (STAGE) {
        const int i0 = (tile % G.ntx) * G.tx, j0 = (tile / G.ntx) * G.ty;
#pragma unroll
        for (int u = 0; u < 3; u++) {
            const int q = t + 64 * u, b = q / (3 * G.tx), rem = q - b * 3 * G.tx, a = rem / 3;
            const bool in = b < G.ty && i0 + a < G.nx && j0 + b < G.ny;
            lo[u] = in ? 3 * (a + G.tx * b) + (rem - 3 * a) : 0;
            go[u] = 3 * ((size_t)i0 + (size_t)G.nx * (in ? j0 + b : j0)) + (in ? rem : 0);
        }
    }
    struct Slot {
        Fac f;
        T w[3];
        TD d;
        double z[3];
    } ring[AH];
    const TD *dpl = dp ? dp : (const TD *)wq;  // without dp a load that is not used
    auto fetch = [&](int s, Slot &Q) {
        const int sc = max(s, 0), tl = L.template load_lane<AH == 2>(G, sc);
        Q.f.template load<NT>(Ft + (size_t)sc * Fac::kStride * 64 + tl);
        const T *w = wt + (size_t)sc * 64 + tl;
        Q.w[0] = w[0]; Q.w[1] = w[S]; Q.w[2] = w[2 * S];
        const size_t g = L.cell(G, sc);
        Q.d = dpl[dp ? g : 0];
        if constexpr (ZIN && STAGE) {
            const double *zl = zin + (size_t)min(s + 1 < 0 ? 0 : s + 1, G.nz - 1) * nxy3;  // layer s + 1
#pragma unroll
            for (int u = 0; u < 3; u++) Q.z[u] = zl[go[u]];
        } else if constexpr (ZIN) {
#pragma unroll
            for (int u = 0; u < 3; u++) Q.z[u] = zin[3 * g + u];
        }
    };
    T xp[3] = {0, 0, 0};
    // slots of this lane's layer and of the layer written, both falling by one a step
    int ks = 0, kf = 0;
    if constexpr (STAGE) {
        ks = ((e - L.a - L.b) % D + D) % D;
        kf = (e + 1) % D;
    }
    auto flush = [&](int k, const double *o, const double *z) {
        double *ol = out + (size_t)min(k, G.nz - 1) * nxy3;
        const bool done = k < G.nz;
#pragma unroll
        for (int u = 0; u < 3; u++) {
            if constexpr (ZIN) ol[go[u]] = done ? z[u] + o[u] : z[u];
            else ol[go[u]] = o[u];
        }
    };
    // fl (a constant at each call): write layer s + 1 out
    auto step = [&](int s, const Slot &Q, bool fl) {
        T xx[3], xy[3];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            xx[c] = __shfl(xp[c], px, 64);
            xy[c] = __shfl(xp[c], py, 64);
        }
        double o[3];
        if (STAGE && fl) {
#pragma unroll
            for (int u = 0; u < 3; u++) o[u] = obuf[kf * 192 + lo[u]];
        }
        T A[9], acc[3], y[3], x[3];
        Q.f.block(2, A);
        mv3(A, xx, acc);
        Q.f.block(3, A);
        mv3(A, xy, y); acc[0] = acc[0] + y[0]; acc[1] = acc[1] + y[1]; acc[2] = acc[2] + y[2];
        Q.f.block(1, A);
        mv3(A, xp, y); acc[0] = acc[0] + y[0]; acc[1] = acc[1] + y[1]; acc[2] = acc[2] + y[2];
        Q.f.block(0, A);
        if constexpr (St == ST_F64) {
            y[0] = Q.w[0] - acc[0]; y[1] = Q.w[1] - acc[1]; y[2] = Q.w[2] - acc[2];
            mv3(A, y, x);
        } else {
            mv3(A, acc, y);
            x[0] = Q.w[0] - y[0]; x[1] = Q.w[1] - y[1]; x[2] = Q.w[2] - y[2];
        }
        const bool act = L.active(G, s);
#pragma unroll
        for (int c = 0; c < 3; c++) xp[c] = act ? x[c] : (T)0;
        const double o0 = dp ? (double)Q.d + (double)xp[0] : (double)xp[0];
        if constexpr (STAGE) {
            // (an idle lane's layer k, below 0 or past nz - 1, shares its slot
            // with layer k +- D, which is written out already or still to come)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            double *ob = obuf + ks * 192 + 3 * t;
            ob[0] = o0;
            ob[1] = (double)xp[1];
            ob[2] = (double)xp[2];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (fl) flush(s + 1, o, Q.z);
            ks = ks == 0 ? D - 1 : ks - 1;
            kf = kf == 0 ? D - 1 : kf - 1;
        } else {
            if (act) {
                double *p = out + 3 * L.cell(G, s);
                p[0] = ZIN ? Q.z[0] + o0 : o0;
                p[1] = ZIN ? Q.z[1] + (double)xp[1] : (double)xp[1];
                p[2] = ZIN ? Q.z[2] + (double)xp[2] : (double)xp[2];
            }
        }
    };
    // whole rounds in which no layer is finished yet, then the rest
#pragma unroll
    for (int u = 0; u < AH; u++) fetch(e - u, ring[u]);
    int s0 = e;
    for (; s0 - AH >= G.nz - 2 && s0 + 1 >= 2 * AH; s0 -= AH)
#pragma unroll
        for (int u = 0; u < AH; u++) {
            step(s0 - u, ring[u], false);
            fetch(s0 - u - AH, ring[u]);
        }
    ring_go<AH>(
        s0 + 1, ring, [&](int q, const Slot &Q) { step(s0 - q, Q, true); }, [&](int q, Slot &Q) { fetch(s0 - q, Q); });
    if constexpr (STAGE) {
        // layer 0, complete with the last step
        double o[3], z[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 3; u++) {
            o[u] = obuf[kf * 192 + lo[u]];
            if constexpr (ZIN) z[u] = zin[go[u]];
        }
        flush(0, o, z);
    }
}

template <int St>
__global__ void k_bj_setup(long long n, const double *__restrict__ A, void *__restrict__ einv,
                           int32_t *__restrict__ bad) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    size_t N = (size_t)n;
    double E[9], Ei[9];
    load_blk(A, S_D, N, (int)g, E);
    if (!inv3_gj(E, Ei)) {
        *bad = 1;
        for (int z = 0; z < 9; z++) Ei[z] = 0.0;
    }
    for (int z = 0; z < 9; z++) {
        if constexpr (St == ST_F64) ((double *)einv)[(size_t)z * N + g] = Ei[z];
        else if constexpr (St == ST_F32) ((float *)einv)[(size_t)z * N + g] = (float)Ei[z];
        else ((uint16_t *)einv)[(size_t)z * N + g] = (uint16_t)bf16_bits((float)Ei[z]);
    }
}

// the same from a general BSR matrix (diagonal block located in each row)
template <int St>
__global__ void k_bj_setup_bsr(long long n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                               const double *__restrict__ val, void *__restrict__ einv, int32_t *__restrict__ bad) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    size_t N = (size_t)n;
    int e = rp[g];
    while (e < rp[g + 1] && ci[e] != (int)g) e++;
    double E[9], Ei[9];
    if (e == rp[g + 1]) {
        *bad = 1;
        for (int z = 0; z < 9; z++) Ei[z] = 0.0;
    } else {
        for (int z = 0; z < 9; z++) E[z] = val[9 * (size_t)e + z];
        if (!inv3_gj(E, Ei)) {
            *bad = 1;
            for (int z = 0; z < 9; z++) Ei[z] = 0.0;
        }
    }
    for (int z = 0; z < 9; z++) {
        if constexpr (St == ST_F64) ((double *)einv)[(size_t)z * N + g] = Ei[z];
        else if constexpr (St == ST_F32) ((float *)einv)[(size_t)z * N + g] = (float)Ei[z];
        else ((uint16_t *)einv)[(size_t)z * N + g] = (uint16_t)bf16_bits((float)Ei[z]);
    }
}

template <int St, typename T, typename TD>
__global__ void k_bj_apply(long long n, const void *__restrict__ einv, const double *__restrict__ r,
                           const TD *__restrict__ dp, double *__restrict__ out) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    size_t N = (size_t)n;
    T Ei[9], v[3] = {(T)r[3 * g], (T)r[3 * g + 1], (T)r[3 * g + 2]}, o[3];
    for (int z = 0; z < 9; z++) {
        if constexpr (St == ST_F64) Ei[z] = ((const double *)einv)[(size_t)z * N + g];
        else if constexpr (St == ST_F32) Ei[z] = ((const float *)einv)[(size_t)z * N + g];
        else Ei[z] = bf16_value(((const uint16_t *)einv)[(size_t)z * N + g]);
    }
    mv3(Ei, v, o);
    out[3 * g] = dp ? (double)dp[g] + (double)o[0] : (double)o[0];
    out[3 * g + 1] = (double)o[1];
    out[3 * g + 2] = (double)o[2];
}

int store_of(const bo_cpr *pc) {
    return pc->o.precision == BO_PREC_FP64 ? ST_F64 : pc->o.precision == BO_PREC_FP32 ? ST_F32 : ST_BF16;
}

// ---- the extended grid form: dual porosity and well rows -----------------------
// Block ILU(0) of the whole system ordered tile by tile: a tile's fracture
// cells (wavefront order as above), then their matrix cells, and the well rows
// as one class of their own after every tile (their couplings to the cells
// dropped, like the couplings between tiles).  A matrix cell's only lower
// neighbour is its fracture cell, so its pivot is E_m = A_mm - (A_mf E_f^{-1})
// A_fm, and a fracture cell's only extra upper neighbour is its matrix cell
// (matrix cells exist in the FP64 form only):
//   forward   y_f (tiles),  y_m = r_m - (A_mf E_f^{-1}) y_f
//   backward  x_m = E_m^{-1} y_m,  x_f = E_f^{-1} (y_f - A_fm x_m - sum_stencil A x)
// The term A_fm x_m is taken out of y_f before the tile's backward sweep.

// matrix pivots E_m^{-1} and the coupling blocks A_mf (row N+g, col g) and
// A_fm (row g, col N+g), SoA 9 x N
__global__ void k_dual_pivots(int n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                              const double *__restrict__ v, const double *__restrict__ einv_f,
                              double *__restrict__ einv_m, double *__restrict__ amf, double *__restrict__ afm,
                              int32_t *__restrict__ bad) {
    int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    size_t N = (size_t)n;
    int ef = rp[g];
    while (ef < rp[g + 1] && ci[ef] != n + g) ef++;
    int em = rp[n + g];  // row N+g holds (g, N+g)
    if (ef == rp[g + 1] || rp[n + g + 1] - em != 2 || ci[em] != g || ci[em + 1] != n + g) {
        *bad = 1;
        return;
    }
    double Af[9], Am[9], Amm[9], Ef[9], L[9], t[9], E[9], Ei[9];
    for (int z = 0; z < 9; z++) {
        Af[z] = v[9 * (size_t)ef + z];
        Am[z] = v[9 * (size_t)em + z];
        Amm[z] = v[9 * (size_t)(em + 1) + z];
        Ef[z] = einv_f[(size_t)z * N + g];
    }
    mul3(Am, Ef, L);
    mul3(L, Af, t);
    for (int z = 0; z < 9; z++) E[z] = Amm[z] - t[z];
    if (!inv3_gj(E, Ei)) {
        *bad = 1;
        for (int z = 0; z < 9; z++) Ei[z] = 0.0;
    }
    for (int z = 0; z < 9; z++) {
        einv_m[(size_t)z * N + g] = Ei[z];
        amf[(size_t)z * N + g] = Am[z];
        afm[(size_t)z * N + g] = Af[z];
    }
}

// inverses of the diagonal blocks of rows [r0, r0 + cnt) (the well rows), 9 x cnt
__global__ void k_rows_inv(int r0, int cnt, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                           const double *__restrict__ v, double *__restrict__ out, int32_t *__restrict__ bad) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= cnt) return;
    int r = r0 + q;
    int e = rp[r];
    while (e < rp[r + 1] && ci[e] != r) e++;
    double E[9], Ei[9];
    if (e == rp[r + 1]) {
        *bad = 1;
        for (int z = 0; z < 9; z++) Ei[z] = 0.0;
    } else {
        for (int z = 0; z < 9; z++) E[z] = v[9 * (size_t)e + z];
        if (!inv3_gj(E, Ei)) {
            *bad = 1;
            for (int z = 0; z < 9; z++) Ei[z] = 0.0;
        }
    }
    for (int z = 0; z < 9; z++) out[(size_t)z * cnt + q] = Ei[z];
}

// forward step of the matrix cells and the fracture adjustment, on the FP64
// forward result y_f (slot order): x_m = E_m^{-1}(r_m - A_mf E_f^{-1} y_f)
// into out (the matrix cell's lower factor is A_mf E_f^{-1} and it has no
// upper neighbour), then y_f -= A_fm x_m (the fracture cell's coupling to its
// matrix cell, taken out before the tile's backward sweep)
__global__ void k_dual_forward(int n, const int32_t *__restrict__ slot_of, size_t S, const double *__restrict__ r,
                               const double *__restrict__ einv_m, const double *__restrict__ amf,
                               const double *__restrict__ afm, const double *__restrict__ einv_f,
                               double *__restrict__ wq, double *__restrict__ out) {
    int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    size_t N = (size_t)n;
    size_t q = (size_t)slot_of[g];
    double yf[3] = {wq[q], wq[S + q], wq[2 * S + q]};
    double B[9], wf[3], y[3], v3[3], xm[3];
    for (int z = 0; z < 9; z++) B[z] = einv_f[(size_t)z * N + g];
    mv3(B, yf, wf);
    for (int z = 0; z < 9; z++) B[z] = amf[(size_t)z * N + g];
    mv3(B, wf, y);
    for (int c = 0; c < 3; c++) v3[c] = r[3 * (N + g) + c] - y[c];
    for (int z = 0; z < 9; z++) B[z] = einv_m[(size_t)z * N + g];
    mv3(B, v3, xm);
    for (int c = 0; c < 3; c++) out[3 * (N + g) + c] = xm[c];
    for (int z = 0; z < 9; z++) B[z] = afm[(size_t)z * N + g];
    mv3(B, xm, y);
    wq[q] = yf[0] - y[0];
    wq[S + q] = yf[1] - y[1];
    wq[2 * S + q] = yf[2] - y[2];
}

// well rows: x_r = E_r^{-1} r_r; with zin != NULL out = zin + (x + (dp, 0, 0))
// (dp on the row's own index; zin may be out)
template <typename TD>
__global__ void k_rows_apply(int r0, int cnt, const double *__restrict__ inv, const double *__restrict__ r,
                             double *out, const TD *__restrict__ dp, const double *zin) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= cnt) return;
    size_t R = (size_t)(r0 + q);
    double B[9], v3[3] = {r[3 * R], r[3 * R + 1], r[3 * R + 2]}, o[3];
    for (int z = 0; z < 9; z++) B[z] = inv[(size_t)z * cnt + q];
    mv3(B, v3, o);
    if (dp) o[0] = (double)dp[R] + o[0];
    for (int c = 0; c < 3; c++) out[3 * R + c] = zin ? zin[3 * R + c] + o[c] : o[c];
}

// the backward sweep's output staging: tile_x + tile_y - 1 layers of 64
// cells x 3 doubles when they fit in 32 KB of LDS (tiles of 16x4, 8x8 and
// smaller), else direct writes
constexpr int kStageBytes = 64 * 3 * (int)sizeof(double);
inline int stage_layers(const TileGeom &G) {
    const int D = G.tx + G.ty - 1;
    return D * kStageBytes <= 32768 ? D : 0;
}

// Steps in flight.  The mixed forms' chain is short of loads while every tile has
// a SIMD of its own (1024 tiles): 100x100x50 in BF16, both sweeps, forward / backward
// steps 4/3, 3/3, 2/2: 55.8, 57.2, 62.0 us, 104x104x31 in FP32 35.9, 36.3, 39.5 us;
// with more tiles two are enough (300x300x60 in FP32 449, 449, 442 us).  In FP64 more
// than two only take registers (104x104x31 4/3, 3/3, 2/2: 49.8, 49.0, 47.4 us;
// 300x300x60 794, 769, 742 us; 400x400x100 2148, 2174, 2109 us).  Before the loads
// were static 104x104x31 took 76 us in FP64, 400x400x100 2184.
constexpr int kFewTiles = 1024, kAheadF = 4, kAheadB = 3;
template <int St> bool few_tiles(const TileGeom &G) { return St != ST_F64 && G.ntx * G.nty <= kFewTiles; }
// Factors larger than the last-level cache are read past it: they are gone
// before the next sweep reads them, and leave it to what the products and the
// V-cycle read again (400x400x100 in FP64, both sweeps: 2156 us through it, 2119 past it).
// Factors that stay in part must not be: 100x100x50 in FP64, 155 MB, forward
// sweep 41 us cached and 70 us past the cache.
// What counts is what is read: tiles of 4x4 columns on the same grid store 501 MB of
// which 134 MB are read (104 us cached, 123 us past the cache).
template <int St, bool FWD> bool past_cache(const TileGeom &G) {
    typedef Factors<St, FWD> Fac;
    return tile_bytes_read(G.ntx * G.nty, G.tx, G.ty, G.nz, Fac::kCount, sizeof(typename Fac::Raw)) > kCacheBytes;
}
template <int St, typename T, int AH>
void launch_forward_ah(const TileGeom &G, const void *F, const double *r, T *wq, hipStream_t s) {
    const int nb = G.ntx * G.nty;
    if (past_cache<St, true>(G)) k_ilu_forward<St, T, AH, true><<<nb, 64, 0, s>>>(G, F, r, wq);
    else k_ilu_forward<St, T, AH, false><<<nb, 64, 0, s>>>(G, F, r, wq);
}
template <int St, typename T>
void launch_forward(const TileGeom &G, const void *F, const double *r, T *wq, hipStream_t s) {
    if constexpr (St != ST_F64)
        if (few_tiles<St>(G)) return launch_forward_ah<St, T, kAheadF>(G, F, r, wq, s);
    launch_forward_ah<St, T, 2>(G, F, r, wq, s);
}
template <int St, typename T, typename TD, int AH, bool NT, bool ZIN>
void launch_backward_ah(const TileGeom &G, const void *F, T *wq, const TD *dp, double *out, const double *zin,
                        hipStream_t s) {
    const int nb = G.ntx * G.nty, D = stage_layers(G);
    if (D > 0)
        k_ilu_backward<St, T, TD, AH, NT, ZIN, true><<<nb, 64, D * kStageBytes, s>>>(G, F, wq, dp, out, D, zin);
    else k_ilu_backward<St, T, TD, AH, NT, ZIN, false><<<nb, 64, 0, s>>>(G, F, wq, dp, out, D, zin);
}
template <int St, typename T, typename TD, bool ZIN>
void launch_backward_zin(const TileGeom &G, const void *F, T *wq, const TD *dp, double *out, const double *zin,
                         hipStream_t s) {
    const bool nt = past_cache<St, false>(G);
    if constexpr (St != ST_F64)
        if (few_tiles<St>(G)) {
            if (nt) launch_backward_ah<St, T, TD, kAheadB, true, ZIN>(G, F, wq, dp, out, zin, s);
            else launch_backward_ah<St, T, TD, kAheadB, false, ZIN>(G, F, wq, dp, out, zin, s);
            return;
        }
    if (nt) launch_backward_ah<St, T, TD, 2, true, ZIN>(G, F, wq, dp, out, zin, s);
    else launch_backward_ah<St, T, TD, 2, false, ZIN>(G, F, wq, dp, out, zin, s);
}
template <int St, typename T, typename TD>
void launch_backward(const TileGeom &G, const void *F, T *wq, const TD *dp, double *out, const double *zin,
                     hipStream_t s) {
    if (zin) launch_backward_zin<St, T, TD, true>(G, F, wq, dp, out, zin, s);
    else launch_backward_zin<St, T, TD, false>(G, F, wq, dp, out, zin, s);
}

TileGeom geom(const bo_cpr *pc) {
    TileGeom T;
    T.nx = pc->g.nx; T.ny = pc->g.ny; T.nz = pc->g.nz;
    T.tx = pc->o.tile_x; T.ty = pc->o.tile_y;
    T.ntx = (T.nx + T.tx - 1) / T.tx;
    T.nty = (T.ny + T.ty - 1) / T.ty;
    T.ns = (T.tx - 1) + (T.ty - 1) + T.nz;
    return T;
}

}  // namespace

// Launches the F stage's factorisation on stream s and reads nothing back:
// its singular-pivot flag (pc->fflag) is read by fstage_check, so the
// factorisation can run on a stream of its own beside the AMG setup.
bo_status fstage_launch(bo_cpr *pc, hipStream_t s) {
    long long n = pc->n;
    int st = store_of(pc);
    BO_TRY(pc->fflag.alloc(1));
    int32_t *ff = pc->fflag.p;
    BO_HIP(hipMemsetAsync(ff, 0, sizeof(int32_t), s));
    if (pc->o.ftype == BO_F_ILU_NATURAL) return nat_launch(pc, s);
    if (pc->o.ftype == BO_F_BJ) {
        BO_TRY(pc->einv.alloc(9 * n));  // FP64 size: large enough for every format
        void *E = pc->einv.p;
        if (pc->general) {
            const int32_t *rp = pc->Arp.p, *ci = pc->Aci.p;
            const double *v = pc->Aval.p;
            if (st == ST_F64) k_bj_setup_bsr<ST_F64><<<grid_for(n), kBlock, 0, s>>>(n, rp, ci, v, E, ff);
            else if (st == ST_F32) k_bj_setup_bsr<ST_F32><<<grid_for(n), kBlock, 0, s>>>(n, rp, ci, v, E, ff);
            else k_bj_setup_bsr<ST_BF16><<<grid_for(n), kBlock, 0, s>>>(n, rp, ci, v, E, ff);
        } else if (st == ST_F64) k_bj_setup<ST_F64><<<grid_for(n), kBlock, 0, s>>>(n, pc->A.p, E, ff);
        else if (st == ST_F32) k_bj_setup<ST_F32><<<grid_for(n), kBlock, 0, s>>>(n, pc->A.p, E, ff);
        else k_bj_setup<ST_BF16><<<grid_for(n), kBlock, 0, s>>>(n, pc->A.p, E, ff);
    } else {
        TileGeom T = geom(pc);
        size_t S = (size_t)T.slots();
        const long long N = pc->g.n();
        const bool ext = pc->general;  // the extended grid form (extra matrix / well rows)
        if (ext) {
            // FP32 / BF16 factors: only without matrix cells (the tiles and the
            // well rows; a matrix cell's pivot needs its fracture cell's E^-1 in
            // natural order, which the FP64 chain writes)
            if (st != ST_F64 && pc->ncell > N)
                return fail(BO_ERR_UNSUPPORTED, "F stage: with matrix cells the extended form's ILU is FP64 only");
            if (st == ST_F64) BO_TRY(pc->x_einv_f.alloc(9 * N));
        }
        // factor buffers: FP64 packed (the FP64 form factors in place), or
        // the FP32 / BF16 layout (a float4 or uint2 per quad; sized for
        // float4) beside an FP64 packed copy that the factorisation reads
        const bool f64 = st == ST_F64;
        BO_TRY(pc->ilu_f.alloc(f64 ? S * kPairs : S * kQuads));
        BO_TRY(pc->ilu_b.alloc(f64 ? S * kPairs : S * kQuads));
        if (!f64) {
            BO_TRY(pc->ilu_pf.alloc(S * kPairs));
            BO_TRY(pc->ilu_pb.alloc(S * kPairs));
        }
        double2 *Pf = f64 ? pc->ilu_f.p : pc->ilu_pf.p, *Pb = f64 ? pc->ilu_b.p : pc->ilu_pb.p;
        BO_TRY(pc->ilu_slot.alloc(n));
        if (f64) BO_TRY(pc->ilu_w.alloc(3 * S));
        else BO_TRY(pc->ilu_w32.alloc(3 * S));
        // idle slots are never read by the sweeps: their factors stay unset
        int nb = T.ntx * T.nty;
        if (ext)
            k_ilu_pack_bsr<<<grid_for(T.slots()), kBlock, 0, s>>>(T, pc->Arp.p, pc->Aci.p, pc->Aval.p, Pf, Pb,
                                                                  pc->ilu_slot.p, ff);
        else
            k_ilu_pack<<<nb * ((T.ns + pack_steps(T) - 1) / pack_steps(T)), kBlock, 0, s>>>(T, pc->A.p, Pf, Pb,
                                                                                     pc->ilu_slot.p);
        if (f64)
            k_ilu_chain<ST_F64><<<nb, 64, 0, s>>>(T, Pf, Pb, ff, ext ? pc->x_einv_f.p : nullptr, nullptr, nullptr);
        else if (st == ST_F32)
            k_ilu_chain<ST_F32><<<nb, 64, 0, s>>>(T, Pf, Pb, ff, nullptr, pc->ilu_f.p, pc->ilu_b.p);
        else
            k_ilu_chain<ST_BF16><<<nb, 64, 0, s>>>(T, Pf, Pb, ff, nullptr, pc->ilu_f.p, pc->ilu_b.p);
        if (ext && pc->ncell > N) {
            BO_TRY(pc->x_einv_m.alloc(9 * N));
            BO_TRY(pc->x_amf.alloc(9 * N));
            BO_TRY(pc->x_afm.alloc(9 * N));
            k_dual_pivots<<<grid_for(N), kBlock, 0, s>>>((int)N, pc->Arp.p, pc->Aci.p, pc->Aval.p, pc->x_einv_f.p,
                                                         pc->x_einv_m.p, pc->x_amf.p, pc->x_afm.p, ff);
        }
        if (ext && pc->n > pc->ncell) {
            int cnt = pc->n - pc->ncell;
            BO_TRY(pc->x_einv_w.alloc(9 * (size_t)cnt));
            k_rows_inv<<<grid_for(cnt), kBlock, 0, s>>>(pc->ncell, cnt, pc->Arp.p, pc->Aci.p, pc->Aval.p,
                                                        pc->x_einv_w.p, ff);
        }
    }
    BO_HIP(hipGetLastError());
    return BO_OK;
}

// The F stage's flag, once the work fstage_launch queued is ordered before s.
bo_status fstage_check(bo_cpr *pc, hipStream_t s) {
    int32_t bad = 0;
    HostRead rd{pc->fflag.p, sizeof bad, &bad};
    BO_TRY(host_reads(&rd, 1, s));
    if (bad & 4)
        return fail(BO_ERR_HIP, "F stage: a wait for a neighbouring tile's values expired (natural-order ILU)");
    if (bad & 2)
        return fail(BO_ERR_UNSUPPORTED, "F stage: a cell row's lower blocks are not its -x, -y, -z neighbours");
    if (bad) return fail(BO_ERR_SINGULAR_BLOCK, "F stage: singular 3x3 pivot block");
    return BO_OK;
}

namespace {
template <int St, typename T, typename TD>
bo_status fstage_run(bo_cpr *pc, const double *r, const TD *dp, double *out, T *wq, hipStream_t s,
                     const double *zin = nullptr) {
    long long n = pc->n;
    if (pc->o.ftype == BO_F_BJ) {
        if (zin) return fail(BO_ERR_UNSUPPORTED, "F stage: no accumulating block-Jacobi form");
        k_bj_apply<St, T, TD><<<grid_for(n), kBlock, 0, s>>>(n, pc->einv.p, r, dp, out);
    } else {
        TileGeom G = geom(pc);
        launch_forward<St, T>(G, pc->ilu_f.p, r, wq, s);
        launch_backward<St, T, TD>(G, pc->ilu_b.p, wq, dp, out, zin, s);
    }
    BO_HIP(hipGetLastError());
    return BO_OK;
}
}  // namespace

// out = F(r) (+ Pi_p dp when dp != NULL); r in natural order
bo_status fstage_apply(bo_cpr *pc, const double *r, const double *dp, double *out, hipStream_t s) {
    if (pc->o.ftype == BO_F_ILU_NATURAL) return nat_apply(pc, r, dp, out, s);
    if (pc->general && pc->o.ftype == BO_F_ILU_TILED) {
        // the extended grid form: tiles of fracture cells, then matrix cells,
        // then well rows (FP64, or FP32 / BF16 tile factors without matrix
        // cells; the well rows' inverses stay FP64)
        if (dp) return fail(BO_ERR_INVALID_ARG, "F stage: extended form takes no pressure correction");
        TileGeom G = geom(pc);
        size_t S = (size_t)G.slots();
        const long long N = pc->g.n();
        const int st = store_of(pc);
        if (st != ST_F64) {
            if (st == ST_F32) launch_forward<ST_F32, float>(G, pc->ilu_f.p, r, pc->ilu_w32.p, s);
            else launch_forward<ST_BF16, float>(G, pc->ilu_f.p, r, pc->ilu_w32.p, s);
            if (pc->n > pc->ncell) {
                int cnt = pc->n - pc->ncell;
                k_rows_apply<double><<<grid_for(cnt), kBlock, 0, s>>>(pc->ncell, cnt, pc->x_einv_w.p, r, out, nullptr,
                                                                      nullptr);
            }
            if (st == ST_F32)
                launch_backward<ST_F32, float, double>(G, pc->ilu_b.p, pc->ilu_w32.p, nullptr, out, nullptr, s);
            else launch_backward<ST_BF16, float, double>(G, pc->ilu_b.p, pc->ilu_w32.p, nullptr, out, nullptr, s);
            BO_HIP(hipGetLastError());
            return BO_OK;
        }
        launch_forward<ST_F64, double>(G, pc->ilu_f.p, r, pc->ilu_w.p, s);
        if (pc->ncell > N)
            k_dual_forward<<<grid_for(N), kBlock, 0, s>>>((int)N, pc->ilu_slot.p, S, r, pc->x_einv_m.p, pc->x_amf.p,
                                                          pc->x_afm.p, pc->x_einv_f.p, pc->ilu_w.p, out);
        if (pc->n > pc->ncell) {
            int cnt = pc->n - pc->ncell;
            k_rows_apply<double><<<grid_for(cnt), kBlock, 0, s>>>(pc->ncell, cnt, pc->x_einv_w.p, r, out, nullptr,
                                                                  nullptr);
        }
        launch_backward<ST_F64, double, double>(G, pc->ilu_b.p, pc->ilu_w.p, nullptr, out, nullptr, s);
        BO_HIP(hipGetLastError());
        return BO_OK;
    }
    switch (store_of(pc)) {
    case ST_F64: return fstage_run<ST_F64, double, double>(pc, r, dp, out, pc->ilu_w.p, s);
    case ST_F32: return fstage_run<ST_F32, float, double>(pc, r, dp, out, pc->ilu_w32.p, s);
    default: return fstage_run<ST_BF16, float, double>(pc, r, dp, out, pc->ilu_w32.p, s);
    }
}

// z += F(r) + Pi_p dp in one pass over z (dp may be NULL; FP64 dp with the
// FP64 factors, FP32 dp with the FP32 / BF16 ones), for the tiled ILU of a
// grid and of the extended form without matrix cells with the pressure system
// over all rows; BO_ERR_UNSUPPORTED for the other forms (the caller then adds
// the terms one by one)
bool fstage_acc_ok(const bo_cpr *pc) {
    if (pc->o.ftype != BO_F_ILU_TILED) return false;
    if (!pc->general) return true;
    return pc->has_grid && pc->ncell == pc->g.n() && pc->npr == pc->n;
}
template <typename TD>
bo_status fstage_apply_acc(bo_cpr *pc, const double *r, const TD *dp, double *z, hipStream_t s) {
    if (!fstage_acc_ok(pc)) return fail(BO_ERR_UNSUPPORTED, "F stage: no accumulating form here");
    const int st = store_of(pc);
    if ((st == ST_F64) != std::is_same<TD, double>::value)
        return fail(BO_ERR_INVALID_ARG, "F stage: pressure correction precision does not match the factors");
    TileGeom G = geom(pc);
    if (pc->general && pc->n > pc->ncell) {
        // the well rows first: they read r and write their own rows of z only
        const int cnt = pc->n - pc->ncell;
        k_rows_apply<TD><<<grid_for(cnt), kBlock, 0, s>>>(pc->ncell, cnt, pc->x_einv_w.p, r, z, dp, z);
        BO_HIP(hipGetLastError());
    }
    if (st == ST_F64)
        return fstage_run<ST_F64, double, TD>(pc, r, dp, z, pc->ilu_w.p, s, z);
    if (st == ST_F32) return fstage_run<ST_F32, float, TD>(pc, r, dp, z, pc->ilu_w32.p, s, z);
    return fstage_run<ST_BF16, float, TD>(pc, r, dp, z, pc->ilu_w32.p, s, z);
}
template bo_status fstage_apply_acc<double>(bo_cpr *, const double *, const double *, double *, hipStream_t);
template bo_status fstage_apply_acc<float>(bo_cpr *, const double *, const float *, double *, hipStream_t);

// mixed form with the FP32 pressure correction of the V-cycle
bo_status fstage_apply_f32dp(bo_cpr *pc, const double *r, const float *dp, double *out, hipStream_t s) {
    switch (store_of(pc)) {
    case ST_F32: return fstage_run<ST_F32, float, float>(pc, r, dp, out, pc->ilu_w32.p, s);
    case ST_BF16: return fstage_run<ST_BF16, float, float>(pc, r, dp, out, pc->ilu_w32.p, s);
    default: return fail(BO_ERR_INVALID_ARG, "F stage: FP32 pressure correction in the FP64 form");
    }
}


}  // namespace bo
