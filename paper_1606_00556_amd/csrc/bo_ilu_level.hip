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
constexpr int kCPairs = 16, kFPairs = 14, kBPairs = 19;
struct NatGeom {
    int nx, ny, nz, ntx, nty, ns;
    __host__ __device__ int tiles() const { return ntx * nty; }
    __host__ __device__ size_t cells() const { return (size_t)nx * ny * nz; }
};
// Packed blocks, as double2 pairs in (tile, row, pair, column) order, the columns
// of a tile being those inside the grid (W of them, 64 but at the grid's edge).
// Layer k of column (a, b) belongs to step s = k + a + b and stands in row
// s mod nz: the steps of a column fall on nz different rows, so the lanes of a
// step read one row (1 KB per wavefront load) and every cell has exactly one
// slot: 816 B a cell with the sweeps' vector, on one layer as on a hundred.
// (A row a step would hold nz + 14 rows of 64 columns: 12.6 KB a cell on one
// layer.)
// C, twice 16 pairs a slot: [A_ii | A_i,-z | A_i,-y | A_i,-x | A_-z,i | A_-y,i |
// A_-x,i], the factorisation's input.  The first 16 pairs of all slots stand
// together: the factorisation leaves the unit-lower factors [L_-z | L_-y | L_-x]
// in 14 of them, and the forward sweep's result y goes into the other two (y0, y1
// as a pair; y2 as one run of doubles), so that the sweeps read the part without
// gaps.  Bp, 19 pairs: [E^-1, pad | A_i,+x | A_i,+y | A_i,+z], blocks outside the
// grid zero.
struct NatTile {
    int i0, j0, wx, wy;  // its first column, its columns in x and y
    size_t base;         // cells of the tiles before it
    __device__ NatTile(const NatGeom &G, int I, int J)
        : i0(I * kNt), j0(J * kNt), wx(min(kNt, G.nx - i0)), wy(min(kNt, G.ny - j0)),
          base(((size_t)j0 * G.nx + (size_t)i0 * wy) * G.nz) {}
};
// where lanes without a cell at a step store (never read), behind Bp's slots
constexpr int kSinks = 64;
__device__ __forceinline__ double2 *nat_sink(const NatGeom &G, double2 *Bp, int lane) {
    return Bp + G.cells() * kBPairs + (blockIdx.x % kSinks) * 64 + lane;
}

__global__ void __launch_bounds__(kBlock) k_nat_pack(NatGeom G, const double *__restrict__ A, double2 *__restrict__ C,
                                                     double2 *__restrict__ Bp) {
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x, N = G.cells();
    if (q >= N) return;
    // the tile, row and column of slot q
    const size_t strip = (size_t)G.nx * kNt * G.nz;  // cells of a full row of tiles
    const int J = (int)(q / strip), wy = min(kNt, G.ny - J * kNt);
    const NatTile T(G, (int)(q % strip / ((size_t)kNt * wy * G.nz)), J);
    const int W = T.wx * T.wy, row = (int)((q - T.base) / W), col = (int)((q - T.base) % W);
    const int a = col % T.wx, b = col / T.wx;
    const int i = T.i0 + a, j = T.j0 + b, k0 = (row - a - b) % G.nz, k = k0 < 0 ? k0 + G.nz : k0;
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
    double2 *c = C + (T.base + (size_t)row * W) * kCPairs + col, *d = Bp + (T.base + (size_t)row * W) * kBPairs + col;
#pragma unroll
    for (int p = 0; p < kCPairs; p++) {
        c[p * W] = make_double2(v[2 * p], v[2 * p + 1]);
        c[N * kCPairs + p * W] = make_double2(v[32 + 2 * p], v[33 + 2 * p]);
    }
#pragma unroll
    for (int p = 5; p < kBPairs; p++) d[p * W] = make_double2(u[2 * p], u[2 * p + 1]);
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

// expired (NULL: not asked for): its bit 4 set if the mark of an expired wait was
__global__ void k_nat_hand_init(size_t n, unsigned long long *__restrict__ H, unsigned long long *__restrict__ ctl,
                                unsigned long long empty, int32_t *__restrict__ expired) {
    const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) H[q] = empty;
    if (q == 1 && expired && ctl[1]) atomicOr(expired, 4);
    if (q < 2) ctl[q] = 0;
}

// Handover of the values at a tile's edge.  The sweeps run in steps u with
// mirrored lane coordinates: p = a, q = b, u = s forward, p = 7 - a, q = 7 - b,
// u = ns - 1 - s backward, so that a tile always takes from the sides p = 0 and
// q = 0 and gives from p = 7 and q = 7.  What a tile takes at step u stands in
// row u mod nz of its own places (an edge column's nz steps fall on nz different
// rows): K values of each of the 8 edge cells of the x side, then of the y side,
// then padding up to NW * 64 words, so that a wavefront looks at the whole row
// with NW loads.  A place is written by one lane of the neighbour and read by
// one lane, once a sweep.  It is empty while it holds kEmpty (a
// signalling NaN with a payload no arithmetic produces); the reader polls until
// it holds something else.  The forward and the backward sweep have their own
// places, and each empties the other's behind its own steps (the factorisation
// has the backward sweep's ones emptied by a launch of its own).  Accesses are
// relaxed 64-bit atomics at agent scope (the XCDs' L2s are not coherent with
// each other otherwise); a value is its own flag, so no ordering between
// accesses is needed.  Row nz takes the writes of lanes that have nothing to
// give.
// Tiles are taken from a ticket in dependence order, so a tile only ever
// waits for tiles that workgroups already running hold.  Waiting is bounded:
// a wavefront polls at most `polls` times in all, then goes on with what it has
// (NaN) and marks ctl[1], which stops every later wait of this handle until
// its next setup: the results are NaN, never a hang.  The setup and the solvers
// read the mark (fstage_check, nat_wait_status) and report the expired wait.
constexpr unsigned long long kEmpty = 0x7FF4A3C15E2D9B87ull;
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
constexpr int hand_words(int K) { return (16 * K + 63) / 64; }  // loads per row

// One wavefront's tile and edges, K values per cell.  The cells' values of the
// last step are kept in LDS, [lane][K] with the taken row behind them, so a
// lane reads its x and y neighbours from places found once.
template <int K, bool FWD>
struct NatLane {
    static constexpr int NW = hand_words(K);
    static constexpr int kLds = 64 * K + NW * 64;  // doubles
    int t, ab, W, c;                // ab: first step (in u) of the lane's column, out of reach without one;
                                    // the tile's columns, the lane's number among them (0 without one)
    size_t base;                    // the tile's first slot
    size_t g0;                      // the column's cell in layer 0
    int rx, ry;                     // LDS places of the -/+x and y neighbours' values
    int take[NW], give[NW], gsrc[NW];  // first steps of taking and giving a word (out of reach: never), its LDS source
    unsigned long long *row, *clr;  // this lane's word in row 0 of the own and of the other sweep's places
    unsigned long long *dst[NW];    // this lane's words in the taking tile's row 0
    unsigned long long *ctl, *sink; // sink: this lane's word of the own row nz
    int spin;
    static constexpr int kNever = 1 << 30;
    __device__ NatLane(const NatGeom &G, const int32_t *__restrict__ order, unsigned long long *H,
                       unsigned long long *other, unsigned long long *ctl_, int polls)
        : t(threadIdx.x), ctl(ctl_) {
        unsigned qt = 0;
        if (t == 0) qt = (unsigned)(atomicAdd(ctl, 1ull) % (unsigned long long)G.tiles());
        qt = __builtin_amdgcn_readfirstlane(qt);
        const int tile = __builtin_amdgcn_readfirstlane(order[FWD ? qt : G.tiles() - 1 - qt]);
        const int a = t % kNt, b = t / kNt;
        const int I = tile % G.ntx, J = tile / G.ntx;
        const NatTile T(G, I, J);
        W = T.wx * T.wy;
        base = T.base;
        const int p = FWD ? a : kNt - 1 - a, q = FWD ? b : kNt - 1 - b;
        auto col = [&](int pp, int qq) {  // a column of the grid, by mirrored coordinates
            return I * kNt + (FWD ? pp : kNt - 1 - pp) < G.nx && J * kNt + (FWD ? qq : kNt - 1 - qq) < G.ny;
        };
        ab = col(p, q) ? p + q : kNever;
        c = col(p, q) ? a + T.wx * b : 0;
        g0 = (size_t)(I * kNt + a) + (size_t)G.nx * (J * kNt + b);
        rx = p > 0 ? (FWD ? t - 1 : t + 1) * K : 64 * K + q * K;
        ry = q > 0 ? (FWD ? t - kNt : t + kNt) * K : 64 * K + (8 + p) * K;
        const bool has_tx = FWD ? I > 0 : I + 1 < G.ntx, has_ty = FWD ? J > 0 : J + 1 < G.nty;
        const bool has_gx = FWD ? I + 1 < G.ntx : I > 0, has_gy = FWD ? J + 1 < G.nty : J > 0;
        const int nx_tile = FWD ? tile + 1 : tile - 1, ny_tile = FWD ? tile + G.ntx : tile - G.ntx;
        const size_t pitch = NW * 64;
        auto place = [&](unsigned long long *set, int tl) { return set + (size_t)tl * (G.nz + 1) * pitch + t; };
        row = place(H, tile);
        clr = place(other, tile);
        sink = row + (size_t)G.nz * pitch;
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const int l = t + 64 * w, e = l / (8 * K), o = l / K % 8, z = l % K;  // side, cell, value
            const bool y = e == 1, edge = e < 2;
            take[w] = edge && (y ? has_ty && col(o, 0) : has_tx && col(0, o)) ? o : kNever;
            const int gp = y ? o : kNt - 1, gq = y ? kNt - 1 : o;
            const bool g = edge && (y ? has_gy : has_gx) && col(gp, gq);
            give[w] = g ? o + kNt - 1 : kNever;
            gsrc[w] = (edge ? (FWD ? gp + kNt * gq : kNt - 1 - gp + kNt * (kNt - 1 - gq)) : t) * K + z;
            dst[w] = g ? place(H, y ? ny_tile : nx_tile) + 64 * w : sink + 64 * w;
        }
        spin = hand_get(ctl + 1) ? 0 : polls;
    }
    __device__ __forceinline__ bool active(const NatGeom &G, int u) const {
        return (unsigned)(u - ab) < (unsigned)G.nz;
    }
    // the cell of an active step (cell 0 otherwise)
    __device__ __forceinline__ size_t cell(const NatGeom &G, int u) const {
        const int k = FWD ? u - ab : G.nz - 1 - (u - ab);
        return active(G, u) ? g0 + (size_t)k * ((size_t)G.nx * G.ny) : 0;
    }
    // the lane's column in the slots of step u (column 0 for an idle lane)
    __device__ __forceinline__ int slot(const NatGeom &G, int u) const { return active(G, u) ? c : 0; }
    // first look at a row of places
    __device__ __forceinline__ void look(int r, unsigned long long *h) const {
        const unsigned long long *p = row + (size_t)r * (NW * 64);
#pragma unroll
        for (int w = 0; w < NW; w++) h[w] = hand_get(p + 64 * w);
    }
    // wait for the values of step u in row r (u mod nz), put them behind the
    // lanes' values in LDS (0 where nothing is taken) and empty the other
    // sweep's row
    __device__ __forceinline__ void taken(const NatGeom &G, int u, int r, unsigned long long *h, double *lds) {
        bool need[NW], miss = false;
#pragma unroll
        for (int w = 0; w < NW; w++) {
            need[w] = (unsigned)(u - take[w]) < (unsigned)G.nz;
            miss = miss || (need[w] && h[w] == kEmpty);
        }
        if (__any(miss)) {
            do {
                if (spin <= 0) {
                    if (t == 0) hand_put(ctl + 1, 1ull);
                    break;
                }
                spin--;
                look(r, h);
                miss = false;
#pragma unroll
                for (int w = 0; w < NW; w++) miss = miss || (need[w] && h[w] == kEmpty);
            } while (__any(miss));
        }
        const size_t o = (size_t)r * (NW * 64);
#pragma unroll
        for (int w = 0; w < NW; w++) {
            lds[64 * K + t + 64 * w] = need[w] ? __longlong_as_double((long long)h[w]) : 0.0;
            if (K == 3) hand_put(clr + o + 64 * w, kEmpty);
        }
    }
    // after the lanes' values of step u are in LDS: hand the edges over, into
    // row r = (u - 7) mod nz of the tiles that take them
    __device__ __forceinline__ void given(const NatGeom &G, int u, int r, const double *lds) const {
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const bool g = (unsigned)(u - give[w]) < (unsigned)G.nz;
            unsigned long long *d = g ? dst[w] + (size_t)r * (NW * 64) : sink + 64 * w;
            hand_put(d, hand_bits(lds[gsrc[w]]));
        }
    }
};
// A row number (a step mod nz) that moves with the steps
struct NatRow {
    int r;
    __device__ NatRow(const NatGeom &G, int step) : r(step % G.nz) { r += r < 0 ? G.nz : 0; }
    __device__ __forceinline__ void up(const NatGeom &G) { r = r + 1 == G.nz ? 0 : r + 1; }
    __device__ __forceinline__ void down(const NatGeom &G) { r = r == 0 ? G.nz - 1 : r - 1; }
};
#define WAVE_FENCE() __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront")

// Factorisation: E_i = A_ii - sum over -z, -y, -x of (A_ik E_k^-1) A_ki, one
// wavefront per tile.  Bound by the arithmetic of a step (six 3x3 products and
// an inverse, FP64 without contraction) times the hyperplanes: 99x101x31 0.77 ms
// (8.8 ms with a launch per hyperplane).
__global__ void __launch_bounds__(64, 1) k_nat_tile_factor(NatGeom G, const int32_t *__restrict__ order,
                                                           double2 *__restrict__ C, double2 *__restrict__ Bp,
                                                           unsigned long long *__restrict__ H,
                                                           unsigned long long *__restrict__ ctl, int polls,
                                                           int32_t *__restrict__ bad) {
    typedef NatLane<9, true> Lane;
    __shared__ double lds[Lane::kLds];
    Lane L(G, order, H, H, ctl, polls);
    const int t = L.t, W = L.W;
    const size_t second = G.cells() * kCPairs;
    double2 *const Ct = C + L.base * kCPairs, *const Bt = Bp + L.base * kBPairs, *const sink = nat_sink(G, Bp, t);
    NatRow now(G, 0), ahead(G, 0), gives(G, 1 - kNt);
#pragma unroll
    for (int z = 0; z < 9; z++) lds[9 * t + z] = 0.0;
    struct Slot {
        double v[64];
        unsigned long long h[Lane::NW];
    } R0, R1;
    double Ep[9];
#pragma unroll
    for (int z = 0; z < 9; z++) Ep[z] = 0.0;
    auto fetch = [&](int s, Slot &S) {
        const double2 *c = Ct + (size_t)ahead.r * W * kCPairs + L.slot(G, s);
#pragma unroll
        for (int p = 0; p < kCPairs; p++) {
            const double2 d = c[p * W], e = c[second + p * W];
            S.v[2 * p] = d.x;
            S.v[2 * p + 1] = d.y;
            S.v[32 + 2 * p] = e.x;
            S.v[33 + 2 * p] = e.y;
        }
        L.look(ahead.r, S.h);
        ahead.up(G);
    };
    auto step = [&](int s, Slot &S) {
        L.taken(G, s, now.r, S.h, lds);
        WAVE_FENCE();
        double Ex[9], Ey[9];
#pragma unroll
        for (int z = 0; z < 9; z++) {
            Ex[z] = lds[L.rx + z];
            Ey[z] = lds[L.ry + z];
        }
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
        const bool act = L.active(G, s);
        if (!inv3_gj(E, Ei)) {
            if (act) atomicOr(bad, 1);
#pragma unroll
            for (int z = 0; z < 9; z++) Ei[z] = 0.0;
        }
        Ei[9] = 0.0;
#pragma unroll
        for (int z = 0; z < 9; z++) {
            Ep[z] = act ? Ei[z] : Ep[z];
            lds[9 * t + z] = Ep[z];
        }
        WAVE_FENCE();
        L.given(G, s, gives.r, lds);
        const int w = act ? W : 0;  // an idle lane's results go to its sink
        double2 *c = act ? Ct + (size_t)now.r * W * kCPairs + L.c : sink;
        double2 *d = act ? Bt + (size_t)now.r * W * kBPairs + L.c : sink;
#pragma unroll
        for (int p = 0; p < kFPairs; p++) c[p * w] = make_double2(lw[2 * p], lw[2 * p + 1]);
#pragma unroll
        for (int p = 0; p < 5; p++) d[p * w] = make_double2(Ei[2 * p], Ei[2 * p + 1]);
        now.up(G);
        gives.up(G);
        fetch(s + 2, S);
    };
    fetch(0, R0);
    fetch(1, R1);
    for (int s0 = 0; s0 < G.ns; s0 += 2) {
        step(s0, R0);
        if (s0 + 1 >= G.ns) break;
        step(s0 + 1, R1);
    }
}

// The sweeps: one wavefront per tile without barriers, the factors, the operand
// and a first look at the handed-over values of AH steps in flight, and
// every load and store issued on every path but the poll that follows a look
// that came too early (vector memory operations return in order and are
// counted statically: a store some paths skip, or the poll as a loop around
// the first look, makes each step wait for the loads of the steps ahead too).
// Sums in the row's column order.  Bound by the latency of a step times the
// nx+ny+nz-2 hyperplanes and by the handovers between tiles: 104x104x31, both
// sweeps, 378 us (3.4 ms with a launch per hyperplane, 456 us with a row of slots
// per step).  A look AH steps ahead needs the neighbour that much further ahead,
// so a short ring wins while every tile has a SIMD of its own (378 / 410 / 490 us
// with 2 / 3 / 4 steps); with more tiles than SIMDs the forward sweep takes 4
// (forward / backward steps 2/2, 3/3, 4/3, 4/2: 4.23, 4.54, 4.21, 4.17 ms on
// 400x400x100, 3/3, 4/3, 4/2: 2.94, 2.71, 2.76 ms on 300x300x100; runs differ by 4 %).

// forward: y_i = r_i - sum_{-z,-y,-x} L y, into Y, the pairs of C behind the factors
template <int AH>
__global__ void __launch_bounds__(64, 1) k_nat_tile_forward(NatGeom G, const int32_t *__restrict__ order,
                                                            const double2 *__restrict__ C,
                                                            double2 *__restrict__ Y, double2 *__restrict__ Bp,
                                                            const double *__restrict__ r,
                                                            unsigned long long *__restrict__ H,
                                                            unsigned long long *__restrict__ other,
                                                            unsigned long long *__restrict__ ctl, int polls) {
    typedef NatLane<3, true> Lane;
    __shared__ double lds[Lane::kLds];
    Lane L(G, order, H, other, ctl, polls);
    const int t = L.t, W = L.W;
    const double2 *Ct = C + L.base * kCPairs;
    double2 *const Yt = Y + L.base * kCPairs + (size_t)kFPairs * W, *const sink = nat_sink(G, Bp, t);
    NatRow now(G, 0), ahead(G, 0), gives(G, 1 - kNt);
#pragma unroll
    for (int c = 0; c < 3; c++) lds[3 * t + c] = 0.0;
    struct Slot {
        double f[28], r[3];
        unsigned long long h[1];
    } ring[AH];
    auto fetch = [&](int s, Slot &Q) {
        const double2 *c = Ct + (size_t)ahead.r * W * kCPairs + L.slot(G, s);
#pragma unroll
        for (int p = 0; p < kFPairs; p++) {
            const double2 d = c[p * W];
            Q.f[2 * p] = d.x;
            Q.f[2 * p + 1] = d.y;
        }
        const double *rg = r + 3 * L.cell(G, s);
        Q.r[0] = rg[0]; Q.r[1] = rg[1]; Q.r[2] = rg[2];
        L.look(ahead.r, Q.h);
        ahead.up(G);
    };
    double yp[3] = {0.0, 0.0, 0.0};
    auto step = [&](int s, Slot &Q) {
        L.taken(G, s, now.r, Q.h, lds);
        WAVE_FENCE();
        double yx[3], yy[3], u[3], v[3] = {Q.r[0], Q.r[1], Q.r[2]};
#pragma unroll
        for (int c = 0; c < 3; c++) {
            yx[c] = lds[L.rx + c];
            yy[c] = lds[L.ry + c];
        }
        mv3d(Q.f, yp, u);
        for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
        mv3d(Q.f + 9, yy, u);
        for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
        mv3d(Q.f + 18, yx, u);
        for (int c = 0; c < 3; c++) v[c] = v[c] - u[c];
        const bool act = L.active(G, s);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            yp[c] = act ? v[c] : 0.0;
            lds[3 * t + c] = yp[c];
        }
        double2 *y = Yt + (size_t)now.r * W * kCPairs;
        *(act ? y + L.c : sink) = make_double2(yp[0], yp[1]);
        *(act ? (double *)(y + W) + L.c : (double *)sink) = yp[2];
        WAVE_FENCE();
        L.given(G, s, gives.r, lds);
        now.up(G);
        gives.up(G);
        fetch(s + AH, Q);
    };
#pragma unroll
    for (int u = 0; u < AH; u++) fetch(u, ring[u]);
    for (int s0 = 0; s0 < G.ns; s0 += AH)
#pragma unroll
        for (int u = 0; u < AH; u++) {
            if (s0 + u >= G.ns) return;
            step(s0 + u, ring[u]);
        }
}

// backward: x_i = E_i^-1 (y_i - sum_{+x,+y,+z} A x), out = x + (dp, 0, 0) in
// natural order (dp may be NULL)
template <int AH>
__global__ void __launch_bounds__(64, 1) k_nat_tile_backward(NatGeom G, const int32_t *__restrict__ order,
                                                             const double2 *__restrict__ C, double2 *__restrict__ Bp,
                                                             const double *__restrict__ dp, double *__restrict__ out,
                                                             unsigned long long *__restrict__ H,
                                                             unsigned long long *__restrict__ other,
                                                             unsigned long long *__restrict__ ctl, int polls) {
    typedef NatLane<3, false> Lane;
    __shared__ double lds[Lane::kLds];
    Lane L(G, order, H, other, ctl, polls);
    const int t = L.t, W = L.W, e = G.ns - 1;
    const double2 *Bt = Bp + L.base * kBPairs, *Yt = C + L.base * kCPairs + (size_t)kFPairs * W;
    double2 *const sink = nat_sink(G, Bp, t);
    // rows of the places (by steps u) and of the slots (by steps s = ns - 1 - u)
    NatRow now(G, 0), ahead(G, 0), gives(G, 1 - kNt), from(G, e);
#pragma unroll
    for (int c = 0; c < 3; c++) lds[3 * t + c] = 0.0;
    struct Slot {
        double f[38], y[3], d;
        unsigned long long h[1];
    } ring[AH];
    const double *dpl = dp ? dp : (const double *)C;  // without dp a load that is not used
    auto fetch = [&](int u, Slot &Q) {
        const int cl = L.slot(G, u);
        const double2 *c = Bt + (size_t)from.r * W * kBPairs + cl;
#pragma unroll
        for (int p = 0; p < kBPairs; p++) {
            const double2 d = c[p * W];
            Q.f[2 * p] = d.x;
            Q.f[2 * p + 1] = d.y;
        }
        const double2 *y = Yt + (size_t)from.r * W * kCPairs, y01 = y[cl];
        Q.y[0] = y01.x; Q.y[1] = y01.y; Q.y[2] = ((const double *)(y + W))[cl];
        Q.d = dpl[dp ? L.cell(G, u) : 0];
        L.look(ahead.r, Q.h);
        ahead.up(G);
        from.down(G);
    };
    double xp[3] = {0.0, 0.0, 0.0};
    auto step = [&](int u, Slot &Q) {
        L.taken(G, u, now.r, Q.h, lds);
        WAVE_FENCE();
        double xx[3], xy[3], w[3], v[3] = {Q.y[0], Q.y[1], Q.y[2]};
#pragma unroll
        for (int c = 0; c < 3; c++) {
            xx[c] = lds[L.rx + c];
            xy[c] = lds[L.ry + c];
        }
        mv3d(Q.f + 10, xx, w);
        for (int c = 0; c < 3; c++) v[c] = v[c] - w[c];
        mv3d(Q.f + 19, xy, w);
        for (int c = 0; c < 3; c++) v[c] = v[c] - w[c];
        mv3d(Q.f + 28, xp, w);
        for (int c = 0; c < 3; c++) v[c] = v[c] - w[c];
        mv3d(Q.f, v, w);
        const bool act = L.active(G, u);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            xp[c] = act ? w[c] : 0.0;
            lds[3 * t + c] = xp[c];
        }
        WAVE_FENCE();
        L.given(G, u, gives.r, lds);
        now.up(G);
        gives.up(G);
        double *o = act ? out + 3 * L.cell(G, u) : (double *)sink;
        o[0] = dp ? Q.d + xp[0] : xp[0];
        o[1] = xp[1];
        o[act ? 2 : 0] = xp[2];
        fetch(u + AH, Q);
    };
#pragma unroll
    for (int u = 0; u < AH; u++) fetch(u, ring[u]);
    for (int u0 = 0; u0 <= e; u0 += AH)
#pragma unroll
        for (int u = 0; u < AH; u++) {
            if (u0 + u > e) return;
            step(u0 + u, ring[u]);
        }
}

constexpr int kNatFewTiles = 1024;  // one per SIMD

NatGeom nat_geom(const Grid &g) {
    NatGeom G;
    G.nx = g.nx; G.ny = g.ny; G.nz = g.nz;
    G.ntx = (g.nx + kNt - 1) / kNt;
    G.nty = (g.ny + kNt - 1) / kNt;
    G.ns = g.nz + 2 * (kNt - 1);
    return G;
}

// the handover memory: the factorisation's places (which the sweeps' two sets
// share), then the ticket and the wait-expired mark
size_t nat_hand_words(const NatGeom &G) { return (size_t)G.tiles() * (G.nz + 1) * 64 * hand_words(9); }

// factorisation of a plain grid from the operator's slot arrays
bo_status nat_tile_launch(bo_cpr *pc, hipStream_t s) {
    const NatGeom G = nat_geom(pc->g);
    const size_t N = G.cells(), nh = nat_hand_words(G);
    BO_TRY(pc->nat_c.alloc(2 * N * kCPairs));
    BO_TRY(pc->nat_b.alloc(N * kBPairs + kSinks * 64));
    BO_TRY(pc->nat_hand.alloc(nh + 2));
    BO_TRY(pc->nat_perm.alloc(G.tiles()));
    unsigned long long *H = pc->nat_hand.p, *ctl = H + nh;
    k_nat_pack<<<grid_for((long long)N), kBlock, 0, s>>>(G, pc->A.p, pc->nat_c.p, pc->nat_b.p);
    k_nat_order<<<grid_for(G.tiles()), kBlock, 0, s>>>(G.ntx, G.nty, pc->nat_perm.p);
    k_nat_hand_init<<<grid_for((long long)nh), kBlock, 0, s>>>(nh, H, ctl, kEmpty, nullptr);
    k_nat_tile_factor<<<G.tiles(), 64, 0, s>>>(G, pc->nat_perm.p, pc->nat_c.p, pc->nat_b.p, H, ctl, pc->nat_polls,
                                               pc->fflag.p);
    k_nat_hand_init<<<grid_for((long long)nh), kBlock, 0, s>>>(nh, H, ctl, kEmpty, pc->fflag.p);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status nat_tile_apply(bo_cpr *pc, const double *r, const double *dp, double *out, hipStream_t s) {
    const NatGeom G = nat_geom(pc->g);
    unsigned long long *H = pc->nat_hand.p, *ctl = H + nat_hand_words(G);
    unsigned long long *Hb = H + nat_hand_words(G) / hand_words(9);  // one word per lane and row for each sweep
    const bool few = G.tiles() <= kNatFewTiles;
    (few ? k_nat_tile_forward<2> : k_nat_tile_forward<4>)<<<G.tiles(), 64, 0, s>>>(
        G, pc->nat_perm.p, pc->nat_c.p, pc->nat_c.p, pc->nat_b.p, r, H, Hb, ctl, pc->nat_polls);
    k_nat_tile_backward<2><<<G.tiles(), 64, 0, s>>>(
        G, pc->nat_perm.p, pc->nat_c.p, pc->nat_b.p, dp, out, Hb, H, ctl, pc->nat_polls);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

}  // namespace

// Factorisation on stream s; it reads nothing back: the flag pc->fflag (bit 1: a
// missing or singular pivot block; bit 2: a cell row with a lower block other
// than its -x, -y, -z neighbours; bit 4: an expired wait of the plain grid's
// kernels) is read by fstage_check.  Grid with well rows: over the handle's BSR
// copy (Arp, Aci, Aval).
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

// BO_ERR_HIP if a wait of an application since the last setup has expired (one
// read of the mark, ordered after the work on s); BO_OK for any other handle
bo_status nat_wait_status(bo_cpr *pc, hipStream_t s) {
    if (pc->bs != 3 || pc->o.ftype != BO_F_ILU_NATURAL || pc->general || !pc->nat_hand.p) return BO_OK;
    uint64_t mark = 0;
    const HostRead rd{pc->nat_hand.p + nat_hand_words(nat_geom(pc->g)) + 1, sizeof mark, &mark};
    BO_TRY(host_reads(&rd, 1, s));
    return mark ? fail(BO_ERR_HIP, "natural-order ILU: a wait for a neighbouring tile's values expired") : BO_OK;
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
