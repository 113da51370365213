// F stage of CPR (Section 3.2) with block ILU(0) in natural order over the
// whole system, applied by level scheduling: the comparison point of the
// tiled form (which drops the couplings between tiles to run one wavefront
// per tile without grid-wide waits).
//
// Block ILU(0) by its IKJ definition, rows in index order: for each lower
// entry k of row i in ascending column order, L_ik = A_ik E_k^{-1} (with A_ik
// as updated so far), then A_ij -= L_ik A_kj for every later entry j of row i
// that row k also holds; E_i is the updated diagonal block.  Solve: y_i = r_i
// - sum_{k<i} L_ik y_k, then x_i = E_i^{-1} (y_i - sum_{j>i} A_ij x_j) with
// the updated upper blocks.
//
// Schedule: in natural order (x fastest, then y, then z) a grid cell's lower
// entries are its -x, -y and -z neighbours, all on the hyperplane i+j+k-1, so
// the cells of one hyperplane depend only on earlier hyperplanes.
//
// Plain grid: the grid is cut into tiles of 8x8 columns, one wavefront each;
// lane (a, b) handles layer k = s - a - b at step s, so inside a tile the
// hyperplanes advance in registers, and the values that cross a tile edge are
// handed over through memory as soon as they exist (see Handover below).  The
// whole sweep is one launch whose critical path is the nx+ny+nz-2
// hyperplanes at the latency of a step, not of a launch.
//
// Grid with further rows (fixed-rate wells): these come after every cell in
// natural order and may couple to each other, and a cell row may hold blocks
// towards them.  The factorisation and each sweep take the hyperplanes one
// launch at a time, one thread per cell, and one thread takes the further rows
// in order after the last hyperplane (before the first one in the backward
// sweep).  Each thread reads its own row's blocks (72 contiguous bytes each)
// and writes its own row only.
#include "bo_cpr.hpp"

namespace bo {
namespace {

// cells (i, j, k) of the grid with i + j + k = l in layer k
__host__ __device__ inline int nat_layer_count(int l, int k, int nx, int ny) {
    const int t = l - k;  // i + j
    if (t < 0) return 0;
    const int jlo = t - (nx - 1) > 0 ? t - (nx - 1) : 0;
    const int jhi = t < ny - 1 ? t : ny - 1;
    return jhi >= jlo ? jhi - jlo + 1 : 0;
}

// the pattern: bit 2 for a cell row whose lower entries are not among its
// -x, -y, -z neighbours, bit 1 for a row without its diagonal block
__global__ void k_nat_check(int n, int N, int nx, int ny, const int32_t *__restrict__ rp,
                            const int32_t *__restrict__ ci, int32_t *bad) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int i = r % nx, j = (r / nx) % ny, k = r / (nx * ny);
    bool diag = false, ok = true;
    for (int e = rp[r]; e < rp[r + 1]; e++) {
        const int c = ci[e];
        if (c == r) diag = true;
        else if (c < r && r < N)
            ok = ok && ((i > 0 && c == r - 1) || (j > 0 && c == r - nx) || (k > 0 && c == r - nx * ny));
    }
    if (!ok) atomicOr(bad, 2);
    if (!diag) atomicOr(bad, 1);
}

// perm[lptr[l] + q] = the q-th cell of hyperplane l, by layer and then by j
__global__ void k_nat_perm(int nx, int ny, int nz, const int32_t *__restrict__ lptr, int32_t *__restrict__ perm) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nx * ny * nz) return;
    const int i = c % nx, j = (c / nx) % ny, k = c / (nx * ny);
    const int l = i + j + k;
    int pos = lptr[l];
    for (int q = 0; q < k; q++) pos += nat_layer_count(l, q, nx, ny);
    const int t = l - k;
    pos += j - (t - (nx - 1) > 0 ? t - (nx - 1) : 0);
    perm[pos] = c;
}

__device__ __forceinline__ void ld9(const double *p, double *a) {
#pragma unroll
    for (int z = 0; z < 9; z++) a[z] = p[z];
}

__device__ __forceinline__ void mv3d(const double *A, const double *x, double *y) {
    y[0] = A[0] * x[0] + A[1] * x[1] + A[2] * x[2];
    y[1] = A[3] * x[0] + A[4] * x[1] + A[5] * x[2];
    y[2] = A[6] * x[0] + A[7] * x[1] + A[8] * x[2];
}

// IKJ elimination of row r over finished rows; false for a missing or
// singular pivot
__device__ bool nat_factor_row(int r, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci, double *lu,
                               double *inv) {
    const int e0 = rp[r], e1 = rp[r + 1];
    int ed = -1;
    for (int e = e0; e < e1; e++) {
        const int k = ci[e];
        if (k == r) ed = e;
        if (k >= r) continue;
        double A[9], Ek[9], L[9];
        ld9(lu + 9 * (size_t)e, A);
        ld9(inv + 9 * (size_t)k, Ek);
        mul3(A, Ek, L);
#pragma unroll
        for (int z = 0; z < 9; z++) lu[9 * (size_t)e + z] = L[z];
        const int f0 = rp[k], f1 = rp[k + 1];
        for (int ej = e + 1; ej < e1; ej++) {
            const int j = ci[ej];
            for (int f = f0; f < f1; f++) {
                const int cf = ci[f];
                if (cf > j) break;
                if (cf != j) continue;
                double U[9], t[9];
                ld9(lu + 9 * (size_t)f, U);
                mul3(L, U, t);
#pragma unroll
                for (int z = 0; z < 9; z++) lu[9 * (size_t)ej + z] = lu[9 * (size_t)ej + z] - t[z];
                break;
            }
        }
    }
    double E[9], Ei[9];
    bool ok = ed >= 0;
    if (ok) {
        ld9(lu + 9 * (size_t)ed, E);
        ok = inv3_gj(E, Ei);
    }
    if (!ok)
        for (int z = 0; z < 9; z++) Ei[z] = 0.0;
#pragma unroll
    for (int z = 0; z < 9; z++) inv[9 * (size_t)r + z] = Ei[z];
    return ok;
}

// one hyperplane of the factorisation (rows perm[0..cnt))
__global__ void k_nat_factor(int cnt, const int32_t *__restrict__ perm, const int32_t *__restrict__ rp,
                             const int32_t *__restrict__ ci, double *lu, double *inv, int32_t *bad) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cnt) return;
    if (!nat_factor_row(perm[t], rp, ci, lu, inv)) atomicOr(bad, 1);
}

// rows [r0, r1) one after the other (one thread)
__global__ void k_nat_factor_seq(int r0, int r1, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                 double *lu, double *inv, int32_t *bad) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    for (int r = r0; r < r1; r++)
        if (!nat_factor_row(r, rp, ci, lu, inv)) atomicOr(bad, 1);
}

// y_r = r_r - sum_{k<r} L_rk y_k (entries in ascending column order)
__device__ __forceinline__ void nat_forward_row(int r, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                                const double *__restrict__ lu, const double *__restrict__ rhs,
                                                double *y) {
    double s[3] = {rhs[3 * (size_t)r], rhs[3 * (size_t)r + 1], rhs[3 * (size_t)r + 2]};
    for (int e = rp[r]; e < rp[r + 1]; e++) {
        const int k = ci[e];
        if (k >= r) break;
        double L[9], yk[3] = {y[3 * (size_t)k], y[3 * (size_t)k + 1], y[3 * (size_t)k + 2]}, t[3];
        ld9(lu + 9 * (size_t)e, L);
        mv3d(L, yk, t);
        for (int q = 0; q < 3; q++) s[q] = s[q] - t[q];
    }
    for (int q = 0; q < 3; q++) y[3 * (size_t)r + q] = s[q];
}

// x_r = E_r^{-1} (y_r - sum_{j>r} U_rj x_j)
__device__ __forceinline__ void nat_backward_row(int r, const int32_t *__restrict__ rp,
                                                 const int32_t *__restrict__ ci, const double *__restrict__ lu,
                                                 const double *__restrict__ inv, const double *__restrict__ y,
                                                 double *x) {
    double s[3] = {y[3 * (size_t)r], y[3 * (size_t)r + 1], y[3 * (size_t)r + 2]};
    for (int e = rp[r]; e < rp[r + 1]; e++) {
        const int j = ci[e];
        if (j <= r) continue;
        double U[9], xj[3] = {x[3 * (size_t)j], x[3 * (size_t)j + 1], x[3 * (size_t)j + 2]}, t[3];
        ld9(lu + 9 * (size_t)e, U);
        mv3d(U, xj, t);
        for (int q = 0; q < 3; q++) s[q] = s[q] - t[q];
    }
    double Ei[9], o[3];
    ld9(inv + 9 * (size_t)r, Ei);
    mv3d(Ei, s, o);
    for (int q = 0; q < 3; q++) x[3 * (size_t)r + q] = o[q];
}

__global__ void k_nat_forward(int cnt, const int32_t *__restrict__ perm, const int32_t *__restrict__ rp,
                              const int32_t *__restrict__ ci, const double *__restrict__ lu,
                              const double *__restrict__ rhs, double *y) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < cnt) nat_forward_row(perm[t], rp, ci, lu, rhs, y);
}

__global__ void k_nat_forward_seq(int r0, int r1, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                  const double *__restrict__ lu, const double *__restrict__ rhs, double *y) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    for (int r = r0; r < r1; r++) nat_forward_row(r, rp, ci, lu, rhs, y);
}

__global__ void k_nat_backward(int cnt, const int32_t *__restrict__ perm, const int32_t *__restrict__ rp,
                               const int32_t *__restrict__ ci, const double *__restrict__ lu,
                               const double *__restrict__ inv, const double *__restrict__ y, double *x) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < cnt) nat_backward_row(perm[t], rp, ci, lu, inv, y, x);
}

// rows r1-1 down to r0 (one thread)
__global__ void k_nat_backward_seq(int r0, int r1, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                   const double *__restrict__ lu, const double *__restrict__ inv,
                                   const double *__restrict__ y, double *x) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    for (int r = r1 - 1; r >= r0; r--) nat_backward_row(r, rp, ci, lu, inv, y, x);
}

// out_r += (dp_r, 0, 0) for the pressure rows
__global__ void k_nat_add_p(int npr, const double *__restrict__ dp, double *out) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < npr) out[3 * (size_t)r] = dp[r] + out[3 * (size_t)r];
}

// ---- plain grid: tiles of 8x8 columns with handed-over edges ----------------------
constexpr int kNt = 8;                    // columns of a tile in x and in y
constexpr int kCPairs = 32, kFPairs = 14, kBPairs = 19;
struct NatGeom {
    int nx, ny, nz, ntx, nty, ns, M;
    __host__ __device__ int tiles() const { return ntx * nty; }
    __host__ __device__ size_t slots() const { return (size_t)ntx * nty * ns * 64; }
    __host__ __device__ size_t hand() const { return (size_t)ntx * nty * M * kNt; }  // cells per direction
};
// Packed blocks, as double2 pairs in (tile, step, pair, lane) order (1 KB per
// wavefront load).  C, 32 pairs a slot: [A_ii | A_i,-z | A_i,-y | A_i,-x |
// A_-z,i | A_-y,i | A_-x,i], the factorisation's input; it leaves the unit-lower
// factors [L_-z | L_-y | L_-x] in the first 14 pairs.  Bp, 19 pairs:
// [E^-1, pad | A_i,+x | A_i,+y | A_i,+z], blocks outside the grid zero.
__device__ __forceinline__ size_t c_index(const NatGeom &G, int tile, int s, int lane) {
    return ((size_t)tile * G.ns + s) * kCPairs * 64 + lane;
}
__device__ __forceinline__ size_t b_index(const NatGeom &G, int tile, int s, int lane) {
    return ((size_t)tile * G.ns + s) * kBPairs * 64 + lane;
}

__global__ void __launch_bounds__(kBlock) k_nat_pack(NatGeom G, const double *__restrict__ A, double2 *__restrict__ C,
                                                     double2 *__restrict__ Bp) {
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= G.slots()) return;
    const int t = (int)(q % 64);
    const int s = (int)((q / 64) % G.ns), tile = (int)(q / 64 / G.ns);
    const int a = t % kNt, b = t / kNt;
    const int i = tile % G.ntx * kNt + a, j = tile / G.ntx * kNt + b, k = s - a - b;
    if (i >= G.nx || j >= G.ny || k < 0 || k >= G.nz) return;  // idle slot, never read
    const size_t N = (size_t)G.nx * G.ny * G.nz;
    const int nxy = G.nx * G.ny, g = i + G.nx * j + nxy * k;
    double v[64], u[38];
    auto blk = [&](bool have, int slot, int row, double *o) {
        const double *p = A + (size_t)slot * 9 * N + (have ? row : g);
#pragma unroll
        for (int z = 0; z < 9; z++) o[z] = have ? p[z * N] : 0.0;
    };
    blk(true, S_D, g, v);
    blk(k > 0, S_MZ, g, v + 9);
    blk(j > 0, S_MY, g, v + 18);
    blk(i > 0, S_MX, g, v + 27);
    blk(k > 0, S_PZ, g - nxy, v + 36);
    blk(j > 0, S_PY, g - G.nx, v + 45);
    blk(i > 0, S_PX, g - 1, v + 54);
    v[63] = 0.0;
    blk(i + 1 < G.nx, S_PX, g, u + 10);
    blk(j + 1 < G.ny, S_PY, g, u + 19);
    blk(k + 1 < G.nz, S_PZ, g, u + 28);
    u[37] = 0.0;
    double2 *c = C + c_index(G, tile, s, t), *d = Bp + b_index(G, tile, s, t);
#pragma unroll
    for (int p = 0; p < kCPairs; p++) c[p * 64] = make_double2(v[2 * p], v[2 * p + 1]);
#pragma unroll
    for (int p = 5; p < kBPairs; p++) d[p * 64] = make_double2(u[2 * p], u[2 * p + 1]);
}

// order[q]: the tiles by ascending I + J, then I (each tile after the ones its
// forward dependences reach)
__global__ void k_nat_order(int ntx, int nty, int32_t *__restrict__ order) {
    const int tile = blockIdx.x * blockDim.x + threadIdx.x;
    if (tile >= ntx * nty) return;
    const int I = tile % ntx, J = tile / ntx, d = I + J;
    int pos = 0;
    for (int q = 0; q < d; q++) pos += min(q, ntx - 1) - max(q - (nty - 1), 0) + 1;
    order[pos + I - max(d - (nty - 1), 0)] = tile;
}

__global__ void k_nat_hand_init(size_t n, unsigned long long *__restrict__ H, unsigned long long *__restrict__ ctl,
                                unsigned long long empty) {
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) H[q] = empty;
    if (q < 2) ctl[q] = 0;
}

// Handover of the values at a tile's edge.  Every edge cell has a place of its
// own in H (the x direction first, then the y direction), written by one
// lane and read by one lane.  A place is empty while it holds kEmpty (a
// signalling NaN with a payload no arithmetic produces); the reader polls
// until it holds something else and puts kEmpty back, so every sweep leaves
// all places empty for the next one.  All accesses are relaxed 64-bit atomics
// at agent scope (the tiles' L2s are not coherent with each other otherwise);
// the value is its own flag, so no ordering between accesses is needed.
// Tiles are taken from a ticket in dependence order, so a tile only ever
// waits for tiles that workgroups already running hold.  Waiting is bounded:
// a wavefront polls at most kSpin times in all, then goes on with what it has
// (NaN) and marks ctl[1], which stops every later wait of this handle until
// its next setup: the results are NaN, never a hang.
constexpr unsigned long long kEmpty = 0x7FF4A3C15E2D9B87ull;
constexpr int kSpin = 1 << 21;
__device__ __forceinline__ unsigned long long hand_get(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void hand_put(unsigned long long *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long hand_bits(double v) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    return u == kEmpty ? 0x7FF8000000000000ull : u;  // an input with kEmpty's bits passes on as another NaN
}

// one lane's view of its tile's edges: in the forward direction it takes from
// the tiles at -x and -y and gives to +x and +y, backward the other way round
struct NatLane {
    int t, a, b, tile;
    bool col;                      // a column of the grid
    bool tx, ty, gx, gy;           // takes / gives in x / y
    unsigned long long *Hx_t, *Hy_t, *Hx_g, *Hy_g;  // place of (step offset 0) in each role
    int st, sg;                    // step offsets of taking and giving
    size_t pitch;                  // words between consecutive steps
};
template <int K, bool FWD>
__device__ __forceinline__ NatLane nat_lane(const NatGeom &G, const int32_t *__restrict__ order,
                                            unsigned long long *__restrict__ H, unsigned long long *__restrict__ ctl) {
    NatLane L;
    L.t = threadIdx.x;
    unsigned q = 0;
    if (L.t == 0) q = (unsigned)(atomicAdd(ctl, 1ull) % (unsigned long long)G.tiles());
    q = __builtin_amdgcn_readfirstlane(q);
    L.tile = order[FWD ? q : G.tiles() - 1 - q];
    L.a = L.t % kNt;
    L.b = L.t / kNt;
    const int I = L.tile % G.ntx, J = L.tile / G.ntx;
    L.col = I * kNt + L.a < G.nx && J * kNt + L.b < G.ny;
    const bool mx = I > 0 && L.a == 0, my = J > 0 && L.b == 0;                       // edges towards -x, -y
    const bool px = I + 1 < G.ntx && L.a == kNt - 1, py = J + 1 < G.nty && L.b == kNt - 1;
    L.tx = L.col && (FWD ? mx : px);
    L.ty = L.col && (FWD ? my : py);
    L.gx = L.col && (FWD ? px : mx);
    L.gy = L.col && (FWD ? py : my);
    // an edge's places belong to the tile on its lower side; cell (k, b) of an
    // x edge stands at step m = k + b, lane b, cell (k, a) of a y edge at m =
    // k + a, lane a
    unsigned long long *Hy = H + G.hand() * 9;
    L.pitch = (size_t)kNt * K;
    auto place = [&](unsigned long long *base, int tile, int lane) { return base + ((size_t)tile * G.M * kNt + lane) * K; };
    unsigned long long *own_x = place(H, L.tile, L.b), *own_y = place(Hy, L.tile, L.a);
    unsigned long long *low_x = place(H, I > 0 ? L.tile - 1 : L.tile, L.b), *low_y = place(Hy, J > 0 ? L.tile - G.ntx : L.tile, L.a);
    L.Hx_t = FWD ? low_x : own_x;
    L.Hy_t = FWD ? low_y : own_y;
    L.Hx_g = FWD ? own_x : low_x;
    L.Hy_g = FWD ? own_y : low_y;
    L.st = FWD ? 0 : kNt - 1;      // m = s - st when taking, s - sg when giving
    L.sg = FWD ? kNt - 1 : 0;
    return L;
}
__device__ __forceinline__ bool nat_active(const NatGeom &G, const NatLane &L, int s) {
    const int k = s - L.a - L.b;
    return L.col && k >= 0 && k < G.nz;
}
template <int K>
struct Hand {
    unsigned long long x[K], y[K];
};
// first look at the places of step s (lanes that take nothing look at place 0)
template <int K>
__device__ __forceinline__ void hand_look(const NatGeom &G, const NatLane &L, int s, Hand<K> &h) {
    const bool act = nat_active(G, L, s);
    const size_t o = act ? (size_t)(s - L.st) * L.pitch : 0;
    const unsigned long long *px = L.Hx_t + (L.tx ? o : 0), *py = L.Hy_t + (L.ty ? o : 0);
#pragma unroll
    for (int z = 0; z < K; z++) {
        h.x[z] = hand_get(px + z);
        h.y[z] = hand_get(py + z);
    }
}
// wait until every value the wavefront takes at step s is there, empty the
// places, and leave zeros in the lanes that take nothing
template <int K>
__device__ __forceinline__ void hand_take(const NatGeom &G, const NatLane &L, int s, Hand<K> &h, int &spin,
                                          unsigned long long *__restrict__ ctl) {
    const bool act = nat_active(G, L, s);
    const bool tx = act && L.tx, ty = act && L.ty;
    auto missing = [&]() {
        bool m = false;
#pragma unroll
        for (int z = 0; z < K; z++) m = m || (tx && h.x[z] == kEmpty) || (ty && h.y[z] == kEmpty);
        return m;
    };
    while (__any(missing())) {
        if (spin <= 0) {
            if (L.t == 0) hand_put(ctl + 1, 1ull);
            break;
        }
        spin--;
        hand_look<K>(G, L, s, h);
    }
    const size_t o = act ? (size_t)(s - L.st) * L.pitch : 0;
    if (tx)
#pragma unroll
        for (int z = 0; z < K; z++) hand_put(L.Hx_t + o + z, kEmpty);
    if (ty)
#pragma unroll
        for (int z = 0; z < K; z++) hand_put(L.Hy_t + o + z, kEmpty);
#pragma unroll
    for (int z = 0; z < K; z++) {
        h.x[z] = tx ? h.x[z] : 0ull;
        h.y[z] = ty ? h.y[z] : 0ull;
    }
}
template <int K>
__device__ __forceinline__ void hand_give(const NatLane &L, int s, const double *v) {
    const size_t o = (size_t)(s - L.sg) * L.pitch;
    if (L.gx)
#pragma unroll
        for (int z = 0; z < K; z++) hand_put(L.Hx_g + o + z, hand_bits(v[z]));
    if (L.gy)
#pragma unroll
        for (int z = 0; z < K; z++) hand_put(L.Hy_g + o + z, hand_bits(v[z]));
}
__device__ __forceinline__ double hand_val(unsigned long long u) { return __longlong_as_double((long long)u); }

// Factorisation: E_i = A_ii - sum over -z, -y, -x of (A_ik E_k^-1) A_ki, one
// wavefront per tile, the neighbours' E^-1 from the lanes of the previous step
// or handed over.  Bound by the arithmetic of a step (six 3x3 products and an
// inverse, FP64 without contraction) times the hyperplanes.
__global__ void __launch_bounds__(64, 1) k_nat_tile_factor(NatGeom G, const int32_t *__restrict__ order,
                                                           double2 *__restrict__ C, double2 *__restrict__ Bp,
                                                           unsigned long long *__restrict__ H,
                                                           unsigned long long *__restrict__ ctl,
                                                           int32_t *__restrict__ bad) {
    const NatLane L = nat_lane<9, true>(G, order, H, ctl);
    const int t = L.t;
    int spin = hand_get(ctl + 1) ? 0 : kSpin;
    struct Slot {
        double v[64];
    } R0, R1;
    Hand<9> h;
    double Ep[9];
#pragma unroll
    for (int z = 0; z < 9; z++) Ep[z] = 0.0;
    auto fetch = [&](int s, Slot &S) {
        const int sc = min(s, G.ns - 1);
        // (idle lanes read a lane of the same step that is in the grid's first
        // column or, where that is idle too, memory of the slot array: unused)
        const double2 *c = C + c_index(G, L.tile, sc, nat_active(G, L, sc) ? t : 0);
#pragma unroll
        for (int p = 0; p < kCPairs; p++) {
            const double2 d = c[p * 64];
            S.v[2 * p] = d.x;
            S.v[2 * p + 1] = d.y;
        }
    };
    auto step = [&](int s, const Slot &S) {
        double Ex[9], Ey[9];
#pragma unroll
        for (int z = 0; z < 9; z++) {
            Ex[z] = __shfl(Ep[z], L.a > 0 ? t - 1 : t, 64);
            Ey[z] = __shfl(Ep[z], L.b > 0 ? t - kNt : t, 64);
        }
        hand_take<9>(G, L, s, h, spin, ctl);
#pragma unroll
        for (int z = 0; z < 9; z++) {
            Ex[z] = L.a > 0 ? Ex[z] : hand_val(h.x[z]);
            Ey[z] = L.b > 0 ? Ey[z] : hand_val(h.y[z]);
        }
        if (s + 1 < G.ns) hand_look<9>(G, L, s + 1, h);
        if (!nat_active(G, L, s)) return;
        const double *v = S.v;
        double E[9], lw[28], tmp[9];
#pragma unroll
        for (int z = 0; z < 9; z++) E[z] = v[z];
        // absent neighbours have zero blocks and zero (never NaN) values
        mul3(v + 9, Ep, lw);
        mul3(lw, v + 36, tmp);
#pragma unroll
        for (int z = 0; z < 9; z++) E[z] = E[z] - tmp[z];
        mul3(v + 18, Ey, lw + 9);
        mul3(lw + 9, v + 45, tmp);
#pragma unroll
        for (int z = 0; z < 9; z++) E[z] = E[z] - tmp[z];
        mul3(v + 27, Ex, lw + 18);
        mul3(lw + 18, v + 54, tmp);
#pragma unroll
        for (int z = 0; z < 9; z++) E[z] = E[z] - tmp[z];
        lw[27] = 0.0;
        double Ei[10];
        if (!inv3_gj(E, Ei)) {
            atomicOr(bad, 1);
#pragma unroll
            for (int z = 0; z < 9; z++) Ei[z] = 0.0;
        }
        Ei[9] = 0.0;
        hand_give<9>(L, s, Ei);
        double2 *c = C + c_index(G, L.tile, s, t), *d = Bp + b_index(G, L.tile, s, t);
#pragma unroll
        for (int p = 0; p < kFPairs; p++) c[p * 64] = make_double2(lw[2 * p], lw[2 * p + 1]);
#pragma unroll
        for (int p = 0; p < 5; p++) d[p * 64] = make_double2(Ei[2 * p], Ei[2 * p + 1]);
#pragma unroll
        for (int z = 0; z < 9; z++) Ep[z] = Ei[z];
    };
    hand_look<9>(G, L, 0, h);
    fetch(0, R0);
    int s0 = 0;
    for (; s0 + 2 <= G.ns; s0 += 2) {
        fetch(s0 + 1, R1);
        step(s0, R0);
        fetch(s0 + 2, R0);
        step(s0 + 1, R1);
    }
    if (s0 < G.ns) step(s0, R0);
}

// The sweeps: one wavefront per tile without barriers, the neighbours' values
// by lane shuffles, the factors, the operand and a first look at the handed-over
// values of kNatAhead steps in flight.  Sums in the row's column order.
// Bound by the latency of a step (its products and shuffles, and a poll of
// the other XCD's memory where the neighbour tile is not ahead) times the
// nx+ny+nz-2 hyperplanes; one launch per hyperplane took 9.4 us each.
constexpr int kNatAhead = 3;

// forward: y_i = r_i - sum_{-z,-y,-x} L y, into yq[3][slot]
__global__ void __launch_bounds__(64, 1) k_nat_tile_forward(NatGeom G, const int32_t *__restrict__ order,
                                                            const double2 *__restrict__ C,
                                                            const double *__restrict__ r, double *__restrict__ yq,
                                                            unsigned long long *__restrict__ H,
                                                            unsigned long long *__restrict__ ctl) {
    const NatLane L = nat_lane<3, true>(G, order, H, ctl);
    const int t = L.t;
    int spin = hand_get(ctl + 1) ? 0 : kSpin;
    const size_t S = G.slots();
    const size_t g0 = (size_t)(L.tile % G.ntx * kNt + L.a) + (size_t)G.nx * (L.tile / G.ntx * kNt + L.b);
    struct Slot {
        double f[28], r[3];
        Hand<3> h;
    } ring[kNatAhead];
    auto fetch = [&](int s, Slot &Q) {
        const int sc = min(s, G.ns - 1);
        const bool act = nat_active(G, L, sc);
        const double2 *c = C + c_index(G, L.tile, sc, act ? t : 0);
#pragma unroll
        for (int p = 0; p < kFPairs; p++) {
            const double2 d = c[p * 64];
            Q.f[2 * p] = d.x;
            Q.f[2 * p + 1] = d.y;
        }
        const double *rg = r + 3 * (act ? g0 + (size_t)(sc - L.a - L.b) * G.nx * G.ny : 0);
        Q.r[0] = rg[0]; Q.r[1] = rg[1]; Q.r[2] = rg[2];
        hand_look<3>(G, L, sc, Q.h);
    };
    double yp[3] = {0.0, 0.0, 0.0};
    auto step = [&](int s, Slot &Q) {
        double yx[3], yy[3];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            yx[c] = __shfl(yp[c], L.a > 0 ? t - 1 : t, 64);
            yy[c] = __shfl(yp[c], L.b > 0 ? t - kNt : t, 64);
        }
        hand_take<3>(G, L, s, Q.h, spin, ctl);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            yx[c] = L.a > 0 ? yx[c] : hand_val(Q.h.x[c]);
            yy[c] = L.b > 0 ? yy[c] : hand_val(Q.h.y[c]);
        }
        if (nat_active(G, L, s)) {
            double u[3], v[3] = {Q.r[0], Q.r[1], Q.r[2]};
            if (s - L.a - L.b > 0) {
                mv3d(Q.f, yp, u);
                for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
            }
            mv3d(Q.f + 9, yy, u);
            for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
            mv3d(Q.f + 18, yx, u);
            for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
            for (int c = 0; c < 3; c++) yp[c] = v[c];
            hand_give<3>(L, s, v);
            const size_t q = ((size_t)L.tile * G.ns + s) * 64 + t;
            yq[q] = v[0]; yq[S + q] = v[1]; yq[2 * S + q] = v[2];
        }
        fetch(s + kNatAhead, Q);
    };
#pragma unroll
    for (int u = 0; u < kNatAhead; u++) fetch(u, ring[u]);
    for (int s0 = 0; s0 < G.ns; s0 += kNatAhead)
#pragma unroll
        for (int u = 0; u < kNatAhead; u++)
            if (s0 + u < G.ns) step(s0 + u, ring[u]);
}

// backward: x_i = E_i^-1 (y_i - sum_{+x,+y,+z} A x), out = x + (dp, 0, 0) in
// natural order (dp may be NULL)
__global__ void __launch_bounds__(64, 1) k_nat_tile_backward(NatGeom G, const int32_t *__restrict__ order,
                                                             const double2 *__restrict__ Bp,
                                                             const double *__restrict__ yq,
                                                             const double *__restrict__ dp, double *__restrict__ out,
                                                             unsigned long long *__restrict__ H,
                                                             unsigned long long *__restrict__ ctl) {
    const NatLane L = nat_lane<3, false>(G, order, H, ctl);
    const int t = L.t;
    int spin = hand_get(ctl + 1) ? 0 : kSpin;
    const size_t S = G.slots();
    const size_t g0 = (size_t)(L.tile % G.ntx * kNt + L.a) + (size_t)G.nx * (L.tile / G.ntx * kNt + L.b);
    const bool last_x = L.a == kNt - 1, last_y = L.b == kNt - 1;
    struct Slot {
        double f[38], y[3], d;
        Hand<3> h;
    } ring[kNatAhead];
    auto fetch = [&](int s, Slot &Q) {
        const int sc = max(s, 0);
        const bool act = nat_active(G, L, sc);
        const int tl = act ? t : 0;
        const double2 *c = Bp + b_index(G, L.tile, sc, tl);
#pragma unroll
        for (int p = 0; p < kBPairs; p++) {
            const double2 d = c[p * 64];
            Q.f[2 * p] = d.x;
            Q.f[2 * p + 1] = d.y;
        }
        const size_t q = ((size_t)L.tile * G.ns + sc) * 64 + tl;
        Q.y[0] = yq[q]; Q.y[1] = yq[S + q]; Q.y[2] = yq[2 * S + q];
        Q.d = dp ? dp[act ? g0 + (size_t)(sc - L.a - L.b) * G.nx * G.ny : 0] : 0.0;
        hand_look<3>(G, L, sc, Q.h);
    };
    double xp[3] = {0.0, 0.0, 0.0};
    auto step = [&](int s, Slot &Q) {
        double xx[3], xy[3];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            xx[c] = __shfl(xp[c], last_x ? t : t + 1, 64);
            xy[c] = __shfl(xp[c], last_y ? t : t + kNt, 64);
        }
        hand_take<3>(G, L, s, Q.h, spin, ctl);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            xx[c] = last_x ? hand_val(Q.h.x[c]) : xx[c];
            xy[c] = last_y ? hand_val(Q.h.y[c]) : xy[c];
        }
        if (nat_active(G, L, s)) {
            double u[3], v[3] = {Q.y[0], Q.y[1], Q.y[2]};
            mv3d(Q.f + 10, xx, u);
            for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
            mv3d(Q.f + 19, xy, u);
            for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
            mv3d(Q.f + 28, xp, u);
            for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
            mv3d(Q.f, v, xp);
            hand_give<3>(L, s, xp);
            double *o = out + 3 * (g0 + (size_t)(s - L.a - L.b) * G.nx * G.ny);
            o[0] = dp ? Q.d + xp[0] : xp[0];
            o[1] = xp[1];
            o[2] = xp[2];
        }
        fetch(s - kNatAhead, Q);
    };
    const int e = G.ns - 1;
#pragma unroll
    for (int u = 0; u < kNatAhead; u++) fetch(e - u, ring[u]);
    for (int s0 = e; s0 >= 0; s0 -= kNatAhead)
#pragma unroll
        for (int u = 0; u < kNatAhead; u++)
            if (s0 - u >= 0) step(s0 - u, ring[u]);
}

NatGeom nat_geom(const Grid &g) {
    NatGeom G;
    G.nx = g.nx; G.ny = g.ny; G.nz = g.nz;
    G.ntx = (g.nx + kNt - 1) / kNt;
    G.nty = (g.ny + kNt - 1) / kNt;
    G.ns = g.nz + 2 * (kNt - 1);
    G.M = g.nz + kNt - 1;
    return G;
}

// factorisation of a plain grid from the operator's slot arrays
bo_status nat_tile_launch(bo_cpr *pc, hipStream_t s) {
    const NatGeom G = nat_geom(pc->g);
    const size_t S = G.slots(), nh = 2 * 9 * G.hand();
    BO_TRY(pc->nat_c.alloc(S * kCPairs));
    BO_TRY(pc->nat_b.alloc(S * kBPairs));
    BO_TRY(pc->nat_y.alloc(3 * S));
    BO_TRY(pc->nat_hand.alloc(nh + 2));
    BO_TRY(pc->nat_perm.alloc(G.tiles()));
    unsigned long long *H = pc->nat_hand.p, *ctl = H + nh;
    k_nat_pack<<<grid_for((long long)S), kBlock, 0, s>>>(G, pc->A.p, pc->nat_c.p, pc->nat_b.p);
    k_nat_order<<<grid_for(G.tiles()), kBlock, 0, s>>>(G.ntx, G.nty, pc->nat_perm.p);
    k_nat_hand_init<<<grid_for((long long)nh), kBlock, 0, s>>>(nh, H, ctl, kEmpty);
    k_nat_tile_factor<<<G.tiles(), 64, 0, s>>>(G, pc->nat_perm.p, pc->nat_c.p, pc->nat_b.p, H, ctl, pc->fflag.p);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status nat_tile_apply(bo_cpr *pc, const double *r, const double *dp, double *out, hipStream_t s) {
    const NatGeom G = nat_geom(pc->g);
    unsigned long long *H = pc->nat_hand.p, *ctl = H + 2 * 9 * G.hand();
    k_nat_tile_forward<<<G.tiles(), 64, 0, s>>>(G, pc->nat_perm.p, pc->nat_c.p, r, pc->nat_y.p, H, ctl);
    k_nat_tile_backward<<<G.tiles(), 64, 0, s>>>(G, pc->nat_perm.p, pc->nat_b.p, pc->nat_y.p, dp, out, H, ctl);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

}  // namespace

// Factorisation on stream s over the handle's BSR copy (Arp, Aci, Aval); it
// reads nothing back: the flag pc->fflag (bit 1: a missing or singular
// pivot, bit 2: a cell row with lower entries off its grid neighbours) is
// read by fstage_check.
bo_status nat_launch(bo_cpr *pc, hipStream_t s) {
    const Grid &g = pc->g;
    const int n = pc->n, N = (int)g.n();
    if (!pc->has_grid || pc->ncell != N || n < N)
        return fail(BO_ERR_UNSUPPORTED, "F stage: the natural-order ILU needs a grid without matrix cells");
    if (!pc->general) return nat_tile_launch(pc, s);
    const int nl = g.nx + g.ny + g.nz - 2;
    pc->nat_lptr.assign(nl + 1, 0);
    for (int l = 0; l < nl; l++) {
        int c = 0;
        for (int k = 0; k < g.nz; k++) c += nat_layer_count(l, k, g.nx, g.ny);
        pc->nat_lptr[l + 1] = pc->nat_lptr[l] + c;
    }
    if (pc->nat_lptr[nl] != N) return fail(BO_ERR_INVALID_ARG, "F stage: hyperplane count mismatch");
    const size_t nnzb = (size_t)pc->nnzb;
    BO_TRY(pc->nat_lu.alloc(9 * nnzb));
    BO_TRY(pc->nat_inv.alloc(9 * (size_t)n));
    BO_TRY(pc->nat_y.alloc(3 * (size_t)n));
    BO_TRY(pc->nat_perm.alloc(N));
    BO_TRY(pc->nat_lptr_d.alloc(nl + 1));
    int32_t *ff = pc->fflag.p;
    const int32_t *rp = pc->Arp.p, *ci = pc->Aci.p;
    BO_HIP(hipMemcpyAsync(pc->nat_lptr_d.p, pc->nat_lptr.data(), sizeof(int32_t) * (nl + 1),
                          hipMemcpyHostToDevice, s));
    BO_HIP(hipMemcpyAsync(pc->nat_lu.p, pc->Aval.p, sizeof(double) * 9 * nnzb, hipMemcpyDeviceToDevice, s));
    k_nat_check<<<grid_for(n), kBlock, 0, s>>>(n, N, g.nx, g.ny, rp, ci, ff);
    k_nat_perm<<<grid_for(N), kBlock, 0, s>>>(g.nx, g.ny, g.nz, pc->nat_lptr_d.p, pc->nat_perm.p);
    BO_HIP(hipGetLastError());
    for (int l = 0; l < nl; l++) {
        const int a = pc->nat_lptr[l], cnt = pc->nat_lptr[l + 1] - a;
        k_nat_factor<<<grid_for(cnt), kBlock, 0, s>>>(cnt, pc->nat_perm.p + a, rp, ci, pc->nat_lu.p, pc->nat_inv.p,
                                                      ff);
    }
    if (n > N) k_nat_factor_seq<<<1, 64, 0, s>>>(N, n, rp, ci, pc->nat_lu.p, pc->nat_inv.p, ff);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

// out = F(r) (+ (dp, 0, 0) on the pressure rows when dp != NULL); out may be r
bo_status nat_apply(bo_cpr *pc, const double *r, const double *dp, double *out, hipStream_t s) {
    if (!pc->general) return nat_tile_apply(pc, r, dp, out, s);
    const int n = pc->n, N = (int)pc->g.n();
    const int nl = (int)pc->nat_lptr.size() - 1;
    const int32_t *rp = pc->Arp.p, *ci = pc->Aci.p, *perm = pc->nat_perm.p;
    const double *lu = pc->nat_lu.p, *inv = pc->nat_inv.p;
    double *y = pc->nat_y.p;
    for (int l = 0; l < nl; l++) {
        const int a = pc->nat_lptr[l], cnt = pc->nat_lptr[l + 1] - a;
        k_nat_forward<<<grid_for(cnt), kBlock, 0, s>>>(cnt, perm + a, rp, ci, lu, r, y);
    }
    if (n > N) {
        k_nat_forward_seq<<<1, 64, 0, s>>>(N, n, rp, ci, lu, r, y);
        k_nat_backward_seq<<<1, 64, 0, s>>>(N, n, rp, ci, lu, inv, y, out);
    }
    for (int l = nl - 1; l >= 0; l--) {
        const int a = pc->nat_lptr[l], cnt = pc->nat_lptr[l + 1] - a;
        k_nat_backward<<<grid_for(cnt), kBlock, 0, s>>>(cnt, perm + a, rp, ci, lu, inv, y, out);
    }
    if (dp) k_nat_add_p<<<grid_for(pc->npr), kBlock, 0, s>>>(pc->npr, dp, out);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

}  // namespace bo
