// Basic operations of Section 3.3 (data structures and algorithms) on the GPU: y = alpha A x + beta y (BSR and
// the library's slot layout), y = alpha x + beta y, dot products and norms,
// plus the prefix sums the setup phases need.
//
// Slot layout of a 7-point 3x3-block matrix: val[(s*9 + e)*N + i] holds entry
// e (row-major in the block) of the block of row i in slot s (-z,-y,-x,diag,
// +x,+y,+z).  Consecutive threads own consecutive rows, so every one of the 63
// value streams is read fully coalesced; blocks outside the grid are zero and
// are skipped.
//
// Reductions are deterministic: a fixed grid of workgroups writes per-group
// partial sums in a fixed tree order, and a second one-workgroup kernel adds
// the partials in a fixed order (no device-scope fences in the hot loop).
#include <algorithm>
#include <chrono>
#include "bo_common.hpp"
#include <cstring>
#include "bo_linalg.hpp"

namespace bo {

static thread_local std::string g_err = "no error";
thread_local const bo_allocator *t_alloc = nullptr;
thread_local void *t_alloc_stream = nullptr;

void set_error(const std::string &msg) { g_err = msg; }
bo_status fail(bo_status st, const std::string &msg) {
    g_err = msg;
    return st;
}

bo_status scratch_get(int slot, size_t bytes, void **ptr) {
    static thread_local void *buf[SC_COUNT] = {};
    static thread_local size_t cap[SC_COUNT] = {};
    if (slot < 0 || slot >= SC_COUNT) return fail(BO_ERR_INVALID_ARG, "scratch slot");
    if (bytes > cap[slot]) {
        if (buf[slot]) (void)hipFree(buf[slot]);
        buf[slot] = nullptr;
        cap[slot] = 0;
        size_t want = std::max<size_t>(bytes, 4096);
        hipError_t e = hipMalloc(&buf[slot], want);
        if (e != hipSuccess)
            return fail(BO_ERR_ALLOC, std::string("scratch hipMalloc failed: ") + hipGetErrorString(e));
        cap[slot] = want;
    }
    *ptr = buf[slot];
    return BO_OK;
}

// ---- small device-to-host reads ---------------------------------------------------
// The words of a call's reads, copied by one kernel into pinned host memory,
// then the call's number: the host waits for that word.  A read used to be a
// copy command per item and a stream synchronisation (about 25 us where the
// stream was idle); a setup makes some fifty of them.
constexpr int kMailItems = 4;
constexpr size_t kMail = 4096;     // bytes of the items; the number stands behind them
struct MailItems {
    const uint32_t *src[kMailItems];
    uint32_t words[kMailItems], off[kMailItems];
    int count;
};
struct Mail {
    char *host = nullptr, *dev = nullptr;  // pinned, coherent; the same memory as the device addresses it
    uint32_t seq = 0;
    static constexpr size_t kFlag = kMail;
};
static thread_local Mail t_mail;

// waits until this wavefront's stores are acknowledged
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// by the threads of one workgroup; the items' words first, then the number
__device__ void mail_write(const MailItems &M, char *mail, uint32_t seq) {
    for (int q = 0; q < M.count; q++)
        for (uint32_t w = threadIdx.x; w < M.words[q]; w += blockDim.x)
            __hip_atomic_store((uint32_t *)(mail + M.off[q]) + w,
                               __hip_atomic_load(M.src[q] + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    // the words are written through at system scope; once they are acknowledged
    // the number may follow (a release fence would write back the whole L2)
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store((uint32_t *)(mail + kMail), seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ void k_mail(MailItems M, char *mail, uint32_t seq) { mail_write(M, mail, seq); }

// the items of r as words in the mail buffer (sizes in whole words)
static bo_status mail_items(const HostRead *r, int count, MailItems &M) {
    if (count < 0 || count > kMailItems) return fail(BO_ERR_INVALID_ARG, "host_reads: at most four items");
    size_t off = 0;
    M.count = count;
    for (int q = 0; q < count; q++) {
        if (r[q].bytes % 4 != 0 || off + r[q].bytes > kMail)
            return fail(BO_ERR_INVALID_ARG, "host_reads: whole words, at most 4 KB");
        M.src[q] = (const uint32_t *)r[q].src;
        M.words[q] = (uint32_t)(r[q].bytes / 4);
        M.off[q] = (uint32_t)off;
        off += (r[q].bytes + 15) / 16 * 16;
    }
    if (!t_mail.host) {
        char *host = nullptr, *dev = nullptr;
        hipError_t e = hipHostMalloc((void **)&host, kMail + 64, hipHostMallocCoherent | hipHostMallocMapped);
        if (e == hipSuccess) e = hipHostGetDevicePointer((void **)&dev, host, 0);
        if (e != hipSuccess) {
            if (host) (void)hipHostFree(host);
            return fail(BO_ERR_ALLOC, std::string("the read buffer could not be allocated: ") + hipGetErrorString(e));
        }
        std::memset(host, 0, kMail + 64);
        t_mail.host = host;
        t_mail.dev = dev;
    }
    t_mail.seq++;
    return BO_OK;
}

// waits for the mail of the last mail_items call (its kernel is enqueued on
// s) and hands the items out.  The host polls for up to kPollMs; a longer wait,
// and any error of the stream, goes through hipStreamSynchronize.
static bo_status mail_take(const HostRead *r, int count, const MailItems &M, hipStream_t s) {
    constexpr double kPollMs = 20.0;
    const uint32_t *flag = (const uint32_t *)(t_mail.host + Mail::kFlag);
    auto there = [&] { return __atomic_load_n(flag, __ATOMIC_ACQUIRE) == t_mail.seq; };
    const auto t0 = std::chrono::steady_clock::now();
    bool ok = false;
    while (!(ok = there())) {
        for (int k = 0; k < 64 && !ok; k++) {
            __builtin_ia32_pause();
            ok = there();
        }
        if (ok || std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count() > kPollMs)
            break;
    }
    if (!ok) {
        BO_HIP(hipStreamSynchronize(s));
        if (!there()) return fail(BO_ERR_HIP, "host_reads: the read did not arrive");
    }
    for (int q = 0; q < count; q++) std::memcpy(r[q].dst, t_mail.host + M.off[q], r[q].bytes);
    return BO_OK;
}

bo_status host_reads(const HostRead *r, int count, hipStream_t s) {
    MailItems M;
    BO_TRY(mail_items(r, count, M));
    k_mail<<<1, kBlock, 0, s>>>(M, t_mail.dev, t_mail.seq);
    BO_HIP(hipGetLastError());
    return mail_take(r, count, M, s);
}

// ---- scan ------------------------------------------------------------------
constexpr int kScanBlock = 1024;

__global__ void k_block_sums(const int32_t *in, int n, int32_t *sums) {
    __shared__ int32_t sh[kScanBlock];
    int base = blockIdx.x * kScanBlock;
    int t = threadIdx.x;
    sh[t] = base + t < n ? in[base + t] : 0;
    __syncthreads();
    for (int w = kScanBlock / 2; w > 0; w >>= 1) {
        if (t < w) sh[t] += sh[t + w];
        __syncthreads();
    }
    if (t == 0) sums[blockIdx.x] = sh[0];
}

// exclusive scan of `sums` (nb entries) in one workgroup, sequential chunks
__global__ void k_scan_sums(int32_t *sums, int nb) {
    __shared__ int32_t sh[kScanBlock];
    __shared__ int32_t carry;
    int t = threadIdx.x;
    if (t == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nb; base += kScanBlock) {
        int v = base + t < nb ? sums[base + t] : 0;
        sh[t] = v;
        __syncthreads();
        for (int off = 1; off < kScanBlock; off <<= 1) {
            int a = t >= off ? sh[t - off] : 0;
            __syncthreads();
            sh[t] += a;
            __syncthreads();
        }
        if (base + t < nb) sums[base + t] = carry + sh[t] - v;
        __syncthreads();
        if (t == kScanBlock - 1) carry += sh[t];
        __syncthreads();
    }
}

__global__ void k_scan_apply(const int32_t *in, int n, const int32_t *sums, int32_t *out) {
    __shared__ int32_t sh[kScanBlock];
    int base = blockIdx.x * kScanBlock;
    int t = threadIdx.x;
    int v = base + t < n ? in[base + t] : 0;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {
        int a = t >= off ? sh[t - off] : 0;
        __syncthreads();
        sh[t] += a;
        __syncthreads();
    }
    if (base + t < n) out[base + t] = sums[blockIdx.x] + sh[t] - v;
    if (base + t == n - 1) out[n] = sums[blockIdx.x] + sh[t];
}

// The same in one workgroup for few counts, a run of them per thread: 900 counts
// 13.8 us as three launches, now 3.4 us; up to 8 k counts 3.7 us on average.
constexpr int kScanSmall = 16384;
__global__ void __launch_bounds__(kScanBlock) k_scan_small(const int32_t *__restrict__ in, int n,
                                                           int32_t *__restrict__ out) {
    constexpr int kRun = kScanSmall / kScanBlock;
    __shared__ int32_t part[kScanBlock / 64];
    const int t = threadIdx.x, lane = t % 64, per = (n + kScanBlock - 1) / kScanBlock, i0 = t * per;
    int32_t v[kRun], sum = 0;
#pragma unroll
    for (int k = 0; k < kRun; k++) {
        const bool is = k < per && i0 + k < n;
        v[k] = is ? in[i0 + k] : 0;
        sum += v[k];
    }
    int32_t upto = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t below = __shfl_up(upto, off, 64);
        if (lane >= off) upto += below;
    }
    if (lane == 63) part[t / 64] = upto;
    __syncthreads();
    int32_t at = upto - sum;
    for (int w = 0; w < t / 64; w++) at += part[w];
#pragma unroll
    for (int k = 0; k < kRun; k++) {
        if (k < per && i0 + k < n) out[i0 + k] = at;
        at += v[k];
    }
    if (t == kScanBlock - 1) out[n] = at;
}

int scan_sum_words(int n) { return n > 0 ? (n + kScanBlock - 1) / kScanBlock : 1; }

bo_status scan_counts_async(const int32_t *counts, int32_t *out, int n, int32_t *sums, hipStream_t s) {
    if (n <= 0) {
        BO_HIP(hipMemsetAsync(out, 0, sizeof(int32_t), s));
        return BO_OK;
    }
    if (n <= kScanSmall) {
        k_scan_small<<<1, kScanBlock, 0, s>>>(counts, n, out);
        BO_HIP(hipGetLastError());
        return BO_OK;
    }
    int nb = (n + kScanBlock - 1) / kScanBlock;
    k_block_sums<<<nb, kScanBlock, 0, s>>>(counts, n, sums);
    k_scan_sums<<<1, kScanBlock, 0, s>>>(sums, nb);
    k_scan_apply<<<nb, kScanBlock, 0, s>>>(counts, n, sums, out);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

// The same prefix sum in one pass (scan_counts), the single-pass scan with
// decoupled look-back of Merrill and Garland (2016): a workgroup takes a tile of
// 4096 counts by ticket, publishes the tile's sum, looks back over the sums
// and prefixes of the tiles before it (a wavefront reads 64 of them at a time)
// and publishes its own prefix.  A word holds (call number, state, value), so
// words of earlier calls read as not yet published and nothing is cleared
// between calls; tickets count on from call to call.  A tile waits only for
// tiles whose workgroups took their tickets before it, each of which
// publishes its sum without waiting.  The workgroup that finishes last writes
// the total and the caller's other words into the mail, so the words are free
// for the next call, on whatever stream, once the mail is there.  Three
// launches and a copy per word before.
constexpr int kScanItems = 4, kScanTile = kScanBlock * kScanItems;
enum : uint64_t { SCAN_SUM = 1, SCAN_PREFIX = 2 };
__device__ __forceinline__ uint64_t scan_word(uint32_t call, uint64_t state, int32_t v) {
    return ((uint64_t)(call & 0x3FFFFFFFu) << 34) | (state << 32) | (uint32_t)v;
}
// ctl: [0] tickets taken, [1] workgroups finished (both `first` at the call's start)
__global__ void __launch_bounds__(kScanBlock) k_scan_mail(const int32_t *in, int32_t *out, int n, uint64_t *words,
                                                          uint32_t *ctl, uint32_t first, uint32_t call, MailItems M,
                                                          char *mail, uint32_t seq) {
    __shared__ int32_t wsum[kScanBlock / 64];
    __shared__ int32_t tile_s, prefix_s, last_s;
    const int t = threadIdx.x, lane = t % 64, wave = t / 64;
    if (t == 0) tile_s = (int)(atomicAdd(&ctl[0], 1u) - first);
    __syncthreads();
    const int tile = tile_s, ntiles = (n + kScanTile - 1) / kScanTile;
    const int base = tile * kScanTile + t * kScanItems;
    int32_t v[kScanItems], sum = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; q++) {
        v[q] = base + q < n ? in[base + q] : 0;
        sum += v[q];
    }
    int32_t inc = sum;  // inclusive over the wavefront, then over the workgroup
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t o = __shfl_up(inc, off, 64);
        inc += lane >= off ? o : 0;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kScanBlock / 64; w++) {
        before += w < wave ? wsum[w] : 0;
        total += wsum[w];
    }
    if (wave == 0) {
        int32_t prefix = 0;
        if (tile > 0) {
            if (lane == 0)
                __hip_atomic_store(&words[tile], scan_word(call, SCAN_SUM, total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            for (int end = tile; end > 0; end -= 64) {  // tiles end - 1 downwards, one per lane
                const int j = end - 1 - lane;
                uint64_t w = 0;
                bool need = j >= 0;
                do {
                    if (need) w = __hip_atomic_load(&words[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    need = need && (uint32_t)(w >> 34) != (call & 0x3FFFFFFFu);
                } while (__any(need));
                const bool full = j >= 0 && ((w >> 32) & 3) == SCAN_PREFIX;
                const uint64_t m = __ballot(full);
                const int stop = m ? __ffsll((unsigned long long)m) - 1 : 64;  // the nearest published prefix
                int32_t add = j >= 0 && lane <= stop ? (int32_t)(uint32_t)w : 0;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) add += __shfl_xor(add, off, 64);
                prefix += add;
                if (m) break;
            }
        }
        if (lane == 0) {
            __hip_atomic_store(&words[tile], scan_word(call, SCAN_PREFIX, prefix + total), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            prefix_s = prefix;
        }
    }
    __syncthreads();
    int32_t at = prefix_s + before + inc - sum;
#pragma unroll
    for (int q = 0; q < kScanItems; q++) {
        if (base + q < n) out[base + q] = at;
        at += v[q];
    }
    // out[n] is read by another workgroup below: written through, and there
    // before this workgroup counts as finished
    if (t == 0 && tile == ntiles - 1)
        __hip_atomic_store(out + n, prefix_s + total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    stores_done();
    __syncthreads();
    if (t == 0) last_s = atomicAdd(&ctl[1], 1u) - first == (uint32_t)(ntiles - 1);
    __syncthreads();
    if (last_s) mail_write(M, mail, seq);
}

bo_status scan_counts(const int32_t *counts, int32_t *out, int n, int32_t *total, hipStream_t s,
                      const HostRead *extra, int nextra) {
    if (nextra < 0 || nextra > 3) return fail(BO_ERR_INVALID_ARG, "scan_counts: at most three extra reads");
    HostRead r[4];
    for (int q = 0; q < nextra; q++) r[1 + q] = extra[q];
    if (n <= 0) {
        int32_t z = 0;
        BO_HIP(hipMemcpyAsync(out, &z, sizeof z, hipMemcpyHostToDevice, s));
        if (nextra > 0) {
            BO_TRY(host_reads(r + 1, nextra, s));
        } else {
            BO_HIP(hipStreamSynchronize(s));
        }
        if (total) *total = 0;
        return BO_OK;
    }
    const int nb = (n + kScanTile - 1) / kScanTile;
    // the host thread's words and counters; new memory starts at zero
    struct Work {
        void *mem = nullptr;
        size_t tiles = 0;
        uint32_t call = 0, tickets = 0;
    };
    static thread_local Work W;
    if ((size_t)nb > W.tiles || W.call >= 0x3FFFFFF0u) {
        if (W.mem) (void)hipFree(W.mem);  // (waits for the device)
        const size_t tiles = std::max<size_t>(nb, 1024);
        W = Work{};
        const hipError_t e = hipMalloc(&W.mem, 8 * (tiles + 1));
        if (e != hipSuccess) {
            W.mem = nullptr;
            return fail(BO_ERR_ALLOC, std::string("scan_counts: hipMalloc failed: ") + hipGetErrorString(e));
        }
        BO_HIP(hipMemset(W.mem, 0, 8 * (tiles + 1)));
        BO_HIP(hipDeviceSynchronize());
        W.tiles = tiles;
    }
    int32_t tot = 0;
    r[0] = HostRead{out + n, sizeof tot, &tot};
    MailItems M;
    BO_TRY(mail_items(r, 1 + nextra, M));
    const uint32_t first = W.tickets;
    W.call++;
    W.tickets += (uint32_t)nb;
    k_scan_mail<<<nb, kScanBlock, 0, s>>>(counts, out, n, (uint64_t *)W.mem + 1, (uint32_t *)W.mem, first, W.call, M,
                                          t_mail.dev, t_mail.seq);
    const hipError_t le = hipGetLastError();
    bo_status st = le != hipSuccess ? fail(BO_ERR_HIP, std::string("scan_counts: ") + hipGetErrorString(le))
                                    : mail_take(r, 1 + nextra, M, s);
    if (st != BO_OK) {
        W.tiles = 0;  // the counters may not match the memory: start over with new memory
        return st;
    }
    if (total) *total = tot;
    return BO_OK;
}

// ---- BSR SpMV on the ABI layout ---------------------------------------------
// y = alpha A x + beta y for BS x BS blocks, BS threads per block row, thread r
// forming component r; sums in block order and, within a block, in column
// order.  A workgroup takes 64 consecutive rows: their blocks are one
// contiguous piece of the value array, which goes through LDS in chunks of 64 CH
// blocks (one chunk for rows of up to CH blocks) with 16-byte non-temporal loads,
// each byte read once; the threads' column indices and x entries are in flight
// beside it.  Bound by HBM.  Reading a block's row per thread from global memory
// (k_bsr_spmv_rows) touches each line three times per component and is bound by
// the L1: 312 us for the 1.23 GB of a 197x203x51 grid (3.9 TB/s), here 204 us (6.0
// TB/s; with temporal loads 8 % more, with one contiguous range of rows per XCD
// 13 % more).
// V16: the value array is 16-byte aligned.  CH 7: 7-point rows; 8: shorter rows on
// average among which some are longer, as in a dual-porosity matrix (fracture
// cells 8, matrix cells 2), whose second chunk of 64 blocks cost as much as the
// first: 16 M rows 379 us, 450 with 7; a 7-point grid's 204 us are 206 with 8.
typedef double dvec2 __attribute__((ext_vector_type(2)));
constexpr int kBsrRows = 64;
template <int BS, bool V16, int CH>
__global__ void __launch_bounds__(kBsrRows *BS) k_bsr_spmv(int first, int n, const int32_t *__restrict__ rp,
                                                           const int32_t *__restrict__ ci,
                                                           const double *__restrict__ v, double alpha,
                                                           const double *__restrict__ x, double beta,
                                                           double *__restrict__ y) {
    constexpr int B2 = BS * BS, NT = kBsrRows * BS, KB = 7, kBsrChunk = CH * kBsrRows;
    constexpr int NLD = (kBsrChunk * B2 / 2 + 1 + NT - 1) / NT;  // pairs per thread
    __shared__ __align__(16) double sv[kBsrChunk * B2 + 2];
    // (rows and blocks are counted from r0 and c0: n and the block count may be 2^31 - 1)
    const int t = threadIdx.x, r = t % BS;
    const int r0 = first + blockIdx.x * kBsrRows, r1 = n - r0 > kBsrRows ? r0 + kBsrRows : n;
    const bool row = t / BS < r1 - r0;
    const int i = row ? r0 + t / BS : r1;
    const int e0 = rp[i], e1 = row ? rp[i + 1] : e0;
    const int c_end = rp[r1];
    const double yi = row && beta != 0.0 ? beta * y[(size_t)i * BS + r] : 0.0;
    double s = 0.0;
    for (int c0 = rp[r0], c1; c0 < c_end; c0 = c1) {
        c1 = c_end - c0 > kBsrChunk ? c0 + kBsrChunk : c_end;
        // this row's blocks in the chunk: the first KB columns and x entries
        const int b0 = min(max(e0, c0), c1) - c0, b1 = min(e1, c1) - c0;
        int c[KB];
        double xj[KB][BS];
#pragma unroll
        for (int k = 0; k < KB; k++) c[k] = ci[c0 + min(b0 + k, c1 - c0 - 1)];
        // the chunk's values, from an even position on
        const size_t d0 = (size_t)c0 * B2 & ~(size_t)1, d1 = (size_t)c1 * B2;
        const int np = (int)((d1 - d0 + 1) / 2), skip = (int)((size_t)c0 * B2 - d0);
        double2 ld[NLD];
#pragma unroll
        for (int u = 0; u < NLD; u++) {
            if (u == NLD - 1 && t + NT * u >= np) continue;  // (a chunk is rarely that full)
            const size_t d = d0 + 2 * (size_t)min(t + NT * u, np - 1);
            if (V16 && d + 1 < d1) {
                const dvec2 q = __builtin_nontemporal_load((const dvec2 *)(v + d));
                ld[u] = make_double2(q.x, q.y);
            } else ld[u] = make_double2(v[d], d + 1 < d1 ? v[d + 1] : 0.0);
        }
#pragma unroll
        for (int k = 0; k < KB; k++)
#pragma unroll
            for (int z = 0; z < BS; z++) xj[k][z] = x[(size_t)c[k] * BS + z];
#pragma unroll
        for (int u = 0; u < NLD; u++)
            if (t + NT * u < np) *(double2 *)(sv + 2 * (t + NT * u)) = ld[u];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KB; k++)
            if (b0 + k < b1) {
                const double *a = sv + skip + (b0 + k) * B2 + BS * r;
#pragma unroll
                for (int z = 0; z < BS; z++) s = s + a[z] * xj[k][z];
            }
        for (int e = b0 + KB; e < b1; e++) {  // rows of more than KB blocks
            const double *a = sv + skip + e * B2 + BS * r, *xe = x + (size_t)ci[c0 + e] * BS;
#pragma unroll
            for (int z = 0; z < BS; z++) s = s + a[z] * xe[z];
        }
        __syncthreads();
    }
    if (row) y[(size_t)i * BS + r] = alpha * s + yi;
}

// The same with BS threads a block row reading their blocks from memory: for few
// rows, where a launch takes what its longest chain of loads takes (2 k rows 3.8 us,
// staged 4.1; 20 k rows 4.0 and 5.1; 32 k rows 6.0 and 5.4; with about 5 blocks a row
// 50 k rows 6.4 and 7.4, 128 k 13.2 and 13.6, 200 k 23.5 and 20.4), and for rows
// that fill a chunk badly or many times over (1 M rows of 2 blocks 32 and 60 us,
// 50 k of 27 30 and 40 us, 20 k of 60 34 and 125 us).
template <int BS>
__global__ void __launch_bounds__(kBlock) k_bsr_spmv_rows(int first, int n, const int32_t *__restrict__ rp,
                                                          const int32_t *__restrict__ ci,
                                                          const double *__restrict__ v, double alpha,
                                                          const double *__restrict__ x, double beta,
                                                          double *__restrict__ y) {
    const unsigned t = blockIdx.x * kBlock + threadIdx.x, lr = t / BS;
    if (lr >= (unsigned)(n - first)) return;
    const int i = first + (int)lr, r = (int)(t % BS);
    double s = 0.0;
    const int e1 = rp[i + 1];
    for (int e = rp[i]; e < e1; e++) {
        const double *a = v + (size_t)(BS * BS) * e + BS * r, *xe = x + (size_t)BS * ci[e];
#pragma unroll
        for (int z = 0; z < BS; z++) s = s + a[z] * xe[z];
    }
    double *const yi = y + (size_t)BS * i + r;
    *yi = alpha * s + (beta == 0.0 ? 0.0 : beta * *yi);
}

template <int BS>
bo_status bsr_spmv_launch(int n, int nnzb, const int32_t *rp, const int32_t *ci, const double *v, double alpha,
                          const double *x, double beta, double *y, hipStream_t s) {
    const long long b = nnzb, full = 6LL * n;
    const bool staged = b >= 4LL * n && b < 8LL * n && n > (b > full ? 3 << 13 : 1 << 17);
    const bool v16 = (uintptr_t)v % 16 == 0;
    // a launch holds fewer than 2^32 threads
    constexpr long long kRows = (long long)kBsrRows << 24;
    for (long long r = 0; r < n; r += kRows) {
        const int r0 = (int)r, end = (int)std::min<long long>(n, r + kRows);
        const unsigned nb = grid_for(end - r, kBsrRows);
        constexpr unsigned NT = kBsrRows * BS;
        if (!staged)
            k_bsr_spmv_rows<BS><<<grid_for((long long)BS * (end - r0)), kBlock, 0, s>>>(r0, end, rp, ci, v, alpha, x,
                                                                                       beta, y);
        else if (b > full && v16) k_bsr_spmv<BS, true, 7><<<nb, NT, 0, s>>>(r0, end, rp, ci, v, alpha, x, beta, y);
        else if (b > full) k_bsr_spmv<BS, false, 7><<<nb, NT, 0, s>>>(r0, end, rp, ci, v, alpha, x, beta, y);
        else if (v16) k_bsr_spmv<BS, true, 8><<<nb, NT, 0, s>>>(r0, end, rp, ci, v, alpha, x, beta, y);
        else k_bsr_spmv<BS, false, 8><<<nb, NT, 0, s>>>(r0, end, rp, ci, v, alpha, x, beta, y);
        BO_HIP(hipGetLastError());
    }
    return BO_OK;
}
template bo_status bsr_spmv_launch<2>(int, int, const int32_t *, const int32_t *, const double *, double, const double *,
                                      double, double *, hipStream_t);

// ---- sliced BSR (general operator of the solver) -------------------------------
// the width of each slice: its longest row, or in a stencil slice 7 + the
// most entries a row has beyond its stencil neighbours
// (a wavefront per slice: one lane per row, the maximum by shuffles)
__global__ void k_sell_width(int n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci, SellGrid G,
                             int32_t *__restrict__ width) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x, S = r >> 6;
    int len = 0;
    if (r < n) {
        len = rp[r + 1] - rp[r];
        if (sell_stencil_slice(G, S)) {
            int nb[NSLOT], extra = 0;
            sell_stencil_nbrs(G, r, nb);
            for (int e = rp[r]; e < rp[r + 1]; e++) extra += sell_slot_in(nb, ci[e]) < 0;
            len = NSLOT + extra;
        }
    }
    for (int off = 32; off > 0; off >>= 1) len = max(len, __shfl_xor(len, off, 64));
    if ((threadIdx.x & 63) == 0 && 64 * S < n) width[S] = len;
}

__global__ void k_sell_fill(int n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                            const double *__restrict__ v, const int32_t *__restrict__ soff, SellGrid G,
                            int32_t *__restrict__ sci, double *__restrict__ sv) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    int S = r >> 6, lane = r & 63;
    int k0 = soff[S], K = soff[S + 1] - k0;
    int e0 = rp[r], len = rp[r + 1] - e0;
    // padding (past the row's end, or a stencil position the row lacks): a
    // zero block on the row's own column (in a stencil slice: the column the
    // kernels derive), so its product adds +0 and the x load stays in bounds
    for (int k = 0; k < K; k++) {
        size_t b = (size_t)(k0 + k) * 64 + lane;
        sci[b] = sell_stencil_slice(G, S) && k < NSLOT ? sell_stencil_col(G, r, k, n) : r;
        for (int z = 0; z < 9; z++) sv[((size_t)(k0 + k) * 9 + z) * 64 + lane] = 0.0;
    }
    const bool st = sell_stencil_slice(G, S);
    int nb[NSLOT];
    if (st) sell_stencil_nbrs(G, r, nb);
    int next = st ? NSLOT : 0;
    for (int q = 0; q < len; q++) {
        const int c = ci[e0 + q];
        int k = st ? sell_slot_in(nb, c) : -1;
        if (k < 0) k = next++;
        size_t b = (size_t)(k0 + k) * 64 + lane;
        sci[b] = c;
        for (int z = 0; z < 9; z++) sv[((size_t)(k0 + k) * 9 + z) * 64 + lane] = v[9 * (size_t)(e0 + q) + z];
    }
}

// One row of the sliced layout, W blocks: every index and value load of the
// row is issued before the first product (no load waits on a branch), then
// the x gathers and the sums in block order.
template <int W, bool ST>
__device__ __forceinline__ void sell_row(const int32_t *__restrict__ sci, const double *__restrict__ sv, int k0,
                                         int lane, const SellGrid &G, int r, int n, const double *__restrict__ x,
                                         double &s0, double &s1, double &s2) {
    int c[W];
#pragma unroll
    for (int k = 0; k < W; k++) c[k] = ST && k < NSLOT ? sell_stencil_col(G, r, k, n) : sci[(size_t)(k0 + k) * 64 + lane];
    double e[W][9];
#pragma unroll
    for (int k = 0; k < W; k++)
#pragma unroll
        for (int z = 0; z < 9; z++) e[k][z] = __builtin_nontemporal_load(sv + ((size_t)(k0 + k) * 9 + z) * 64 + lane);
#pragma unroll
    for (int k = 0; k < W; k++) {
        const double *xj = x + 3 * (size_t)c[k];
        double x0 = xj[0], x1 = xj[1], x2 = xj[2];
        s0 = s0 + e[k][0] * x0; s0 = s0 + e[k][1] * x1; s0 = s0 + e[k][2] * x2;
        s1 = s1 + e[k][3] * x0; s1 = s1 + e[k][4] * x1; s1 = s1 + e[k][5] * x2;
        s2 = s2 + e[k][6] * x0; s2 = s2 + e[k][7] * x1; s2 = s2 + e[k][8] * x2;
    }
}

// y = alpha A x + beta y on the sliced layout: the blocks of a row in their
// BSR order and each block's entries in order, as k_bsr_spmv; the 64 lanes of
// a wavefront read each of a block column's 9 value arrays as one 512 B line
// pair (non-temporal: read once per launch).  A wavefront is one slice, so the
// slice width selects one path for all its lanes: widths 7 and 8 (the 7-point
// stencil, and a row with a well block) unrolled, others in a loop.  Padding
// blocks are zero blocks on the row's own column and add +0.
__global__ void __launch_bounds__(kBlock) k_sell_spmv(int n, const int32_t *__restrict__ soff,
                                                      const int32_t *__restrict__ sci,
                                                      const double *__restrict__ sv, SellGrid G, double alpha,
                                                      const double *__restrict__ x, double beta,
                                                      const double *yin, double *y) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    int S = r >> 6, lane = r & 63;
    int k0 = soff[S], K = soff[S + 1] - k0;
    const bool st = sell_stencil_slice(G, S);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (K == 7) {
        if (st) sell_row<7, true>(sci, sv, k0, lane, G, r, n, x, s0, s1, s2);
        else sell_row<7, false>(sci, sv, k0, lane, G, r, n, x, s0, s1, s2);
    } else if (K == 8) {
        if (st) sell_row<8, true>(sci, sv, k0, lane, G, r, n, x, s0, s1, s2);
        else sell_row<8, false>(sci, sv, k0, lane, G, r, n, x, s0, s1, s2);
    } else {
        for (int k = 0; k < K; k++) {
            int c = st && k < NSLOT ? sell_stencil_col(G, r, k, n) : sci[(size_t)(k0 + k) * 64 + lane];
            const double *blk = sv + (size_t)(k0 + k) * 9 * 64 + lane;
            double e[9];
#pragma unroll
            for (int z = 0; z < 9; z++) e[z] = __builtin_nontemporal_load(blk + z * 64);
            double x0 = x[3 * (size_t)c], x1 = x[3 * (size_t)c + 1], x2 = x[3 * (size_t)c + 2];
            s0 = s0 + e[0] * x0; s0 = s0 + e[1] * x1; s0 = s0 + e[2] * x2;
            s1 = s1 + e[3] * x0; s1 = s1 + e[4] * x1; s1 = s1 + e[5] * x2;
            s2 = s2 + e[6] * x0; s2 = s2 + e[7] * x1; s2 = s2 + e[8] * x2;
        }
    }
    // y = alpha A x + beta yin (yin is y itself, or another vector)
    const double *wi = yin + 3 * (size_t)r;
    double t0 = beta == 0.0 ? 0.0 : beta * wi[0];
    double t1 = beta == 0.0 ? 0.0 : beta * wi[1];
    double t2 = beta == 0.0 ? 0.0 : beta * wi[2];
    double *yi = y + 3 * (size_t)r;
    yi[0] = alpha * s0 + t0;
    yi[1] = alpha * s1 + t1;
    yi[2] = alpha * s2 + t2;
}

// r -= A Pi_p dp on the sliced layout, in place: column 0 of each block (3
// of its 9 value arrays), dp on the block columns below npr (0 elsewhere;
// padding blocks sit on the row's own column with zero values).
template <typename TD>
__global__ void __launch_bounds__(kBlock) k_sell_col0_update(int n, int npr, const int32_t *__restrict__ soff,
                                                             const int32_t *__restrict__ sci,
                                                             const double *__restrict__ sv, SellGrid G,
                                                             const TD *__restrict__ dp, double *r) {
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= n) return;
    const int S = row >> 6, lane = row & 63;
    const int k0 = soff[S], K = soff[S + 1] - k0;
    const bool st = sell_stencil_slice(G, S);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int k = 0; k < K; k++) {
        const int c = st && k < NSLOT ? sell_stencil_col(G, row, k, n) : sci[(size_t)(k0 + k) * 64 + lane];
        const double *blk = sv + (size_t)(k0 + k) * 9 * 64 + lane;
        const double p = c < npr ? (double)dp[c] : 0.0;
        s0 = s0 + __builtin_nontemporal_load(blk) * p;
        s1 = s1 + __builtin_nontemporal_load(blk + 3 * 64) * p;
        s2 = s2 + __builtin_nontemporal_load(blk + 6 * 64) * p;
    }
    double *ri = r + 3 * (size_t)row;
    ri[0] = ri[0] - s0;
    ri[1] = ri[1] - s1;
    ri[2] = ri[2] - s2;
}

// r -= A Pi_p dp on the slot layout, in place (column 0 of each block)
template <typename TD>
__global__ void __launch_bounds__(kBlock) k_slot_col0_update(int nx, int ny, int nz, const double *__restrict__ A,
                                                             const TD *__restrict__ dp, double *r) {
    const int n = nx * ny * nz;
    const int i = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const size_t N = (size_t)n;
    const int nxy = nx * ny;
    const int ix = i % nx, iy = (i / nx) % ny, iz = i / nxy;
    const int nb[7] = {iz > 0 ? i - nxy : -1, iy > 0 ? i - nx : -1, ix > 0 ? i - 1 : -1, i,
                       ix < nx - 1 ? i + 1 : -1, iy < ny - 1 ? i + nx : -1, iz < nz - 1 ? i + nxy : -1};
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int q = 0; q < NSLOT; q++) {
        const int j = nb[q];
        if (j < 0) continue;
        const double *a = A + (size_t)q * 9 * N + i;
        const double p = (double)dp[j];
        s0 = s0 + a[0 * N] * p;
        s1 = s1 + a[3 * N] * p;
        s2 = s2 + a[6 * N] * p;
    }
    double *ri = r + 3 * (size_t)i;
    ri[0] = ri[0] - s0;
    ri[1] = ri[1] - s1;
    ri[2] = ri[2] - s2;
}

// quasi-IMPES weights of a cell from its diagonal block D (BS = 3: the 2x2
// saturation block in full or its diagonal; BS = 2: the one saturation entry),
// signed for a positive decoupled diagonal; false for a singular one
template <int BS>
__device__ __forceinline__ bool qi_weights(const double *D, int mode, double *c) {
    bool ok = true;
    double w0 = 0.0, w1 = 0.0, dpp;
    if constexpr (BS == 3) {
        const double a = D[4], b = D[5], cc = D[7], d = D[8], p0 = D[1], p1 = D[2];
        if (mode == BO_QI_DIAG) {
            ok = !(a == 0.0 || d == 0.0);
            if (ok) { w0 = p0 / a; w1 = p1 / d; }
        } else {
            const double det = a * d - b * cc;
            ok = !(det == 0.0 || !isfinite(det));
            if (ok) {
                w0 = (p0 * d - p1 * cc) / det;
                w1 = (p1 * a - p0 * b) / det;
            }
        }
        dpp = D[0] - w0 * D[3] - w1 * D[6];
    } else {
        const double d11 = D[3], d01 = D[1];
        ok = !(d11 == 0.0 || !isfinite(d11));
        if (ok) w0 = d01 / d11;
        dpp = D[0] - w0 * D[2];
    }
    const double sg = dpp < 0.0 ? -1.0 : 1.0;
    c[0] = sg;
    c[1] = -sg * w0;
    if (BS == 3) c[2] = -sg * w1;
    return ok;
}

// A grid's BSR matrix into the handle, in one pass over it: the slot layout,
// the decoupling weights and the decoupled pressure block, with the checks.
// flag: bit 1 a row that is not the 7-point stencil's, bit 2 a value that is
// not finite, bit 4 a singular saturation block.  A workgroup stages the blocks
// of 64 rows (one contiguous piece of at most 448 blocks) in LDS with 16-byte
// loads and writes every slot plane 64 rows at a time.  Bound by HBM (BS = 3:
// 504 B read and 588 B written per cell).  At 500k cells a finiteness pass, one
// thread per row copying its blocks plane by plane and a decoupling pass over
// the planes took 50 + 238 + 37 us, at 2M cells 200 + 924 + 150 us; now 101 and
// 468 us (4.7 TB/s, the rate of a large copy).
constexpr int kStencilChunk = 7 * kBsrRows;
enum { IMP_PATTERN = 1, IMP_NONFINITE = 2, IMP_SINGULAR = 4 };
template <int BS, bool V16>
__global__ void __launch_bounds__(256) k_grid_import(int nx, int ny, int nz, const int32_t *__restrict__ rp,
                                                     const int32_t *__restrict__ ci, const double *__restrict__ v,
                                                     int mode, double *__restrict__ slots, double *__restrict__ cw,
                                                     double *__restrict__ app, int32_t *__restrict__ flag) {
    constexpr int B2 = BS * BS, NT = 256;
    constexpr int NLD = (kStencilChunk * B2 / 2 + 1 + NT - 1) / NT;
    __shared__ __align__(16) double sv[kStencilChunk * B2 + 2];
    __shared__ int first[kBsrRows];  // a row's first block in the chunk
    __shared__ unsigned have[kBsrRows];
    const int n = nx * ny * nz, nxy = nx * ny;
    const size_t N = (size_t)n;
    const int t = threadIdx.x, lr = t % kBsrRows, grp = t / kBsrRows;
    const int r0 = blockIdx.x * kBsrRows, r1 = min(r0 + kBsrRows, n), i = r0 + lr;
    const int c0 = rp[r0], c1 = rp[r1];
    if (c1 < c0 || c1 - c0 > kStencilChunk) {
        if (t == 0) atomicOr(flag, IMP_PATTERN);
        return;
    }
    int bad = 0;
    // the chunk's values, from an even position on
    const size_t d0 = (size_t)c0 * B2 & ~(size_t)1, d1 = (size_t)c1 * B2;
    const int np = (int)((d1 - d0 + 1) / 2), skip = (int)((size_t)c0 * B2 - d0);
    double2 ld[NLD];
#pragma unroll
    for (int u = 0; u < NLD; u++) {
        const int q = t + NT * u;
        const size_t d = d0 + 2 * (size_t)q;
        ld[u] = make_double2(0.0, 0.0);
        if (q < np) {
            if (V16 && d + 1 < d1) {
                const dvec2 w = __builtin_nontemporal_load((const dvec2 *)(v + d));
                ld[u] = make_double2(w.x, w.y);
            } else {
                ld[u] = make_double2(v[d], d + 1 < d1 ? v[d + 1] : 0.0);
            }
        }
    }
    // the pattern, one row per thread of the first wavefront
    if (grp == 0) {
        unsigned m = 0;
        int f = 0;
        if (i < n) {
            const int ix = i % nx, iy = (i / nx) % ny, iz = i / nxy;
            m = (iz > 0 ? 1u << S_MZ : 0u) | (iy > 0 ? 1u << S_MY : 0u) | (ix > 0 ? 1u << S_MX : 0u) | (1u << S_D) |
                (ix + 1 < nx ? 1u << S_PX : 0u) | (iy + 1 < ny ? 1u << S_PY : 0u) | (iz + 1 < nz ? 1u << S_PZ : 0u);
            const int e0 = rp[i], e1 = rp[i + 1];
            f = e0 - c0;
            if (e1 - e0 != __popc(m) || f < 0 || f + __popc(m) > c1 - c0) {
                bad |= IMP_PATTERN;
                m = 0;
            } else {
                const int nb[NSLOT] = {i - nxy, i - nx, i - 1, i, i + 1, i + nx, i + nxy};
#pragma unroll
                for (int s = 0; s < NSLOT; s++)
                    if ((m >> s) & 1u)
                        if (ci[e0 + __popc(m & ((1u << s) - 1u))] != nb[s]) bad |= IMP_PATTERN;
            }
        }
        first[lr] = f;
        have[lr] = m;
    }
#pragma unroll
    for (int u = 0; u < NLD; u++)
        if (t + NT * u < np) {
            if (!isfinite(ld[u].x) || !isfinite(ld[u].y)) bad |= IMP_NONFINITE;
            *(double2 *)(sv + 2 * (t + NT * u)) = ld[u];
        }
    __syncthreads();
    const unsigned m = have[lr];
    const double *row = sv + skip + first[lr] * B2;
    if (i < n) {
        // (a wavefront writes one plane of its 64 rows at a time)
        for (int p = grp; p < NSLOT * B2; p += NT / kBsrRows) {
            const int s = p / B2, z = p % B2;
            const bool h = (m >> s) & 1u;
            slots[(size_t)p * N + i] = h ? row[__popc(m & ((1u << s) - 1u)) * B2 + z] : 0.0;
        }
        if (grp == NT / kBsrRows - 1) {
            double D[B2], c[BS];
#pragma unroll
            for (int z = 0; z < B2; z++) D[z] = m ? row[__popc(m & ((1u << S_D) - 1u)) * B2 + z] : 0.0;
            if (!qi_weights<BS>(D, mode, c)) bad |= IMP_SINGULAR;
#pragma unroll
            for (int z = 0; z < BS; z++) cw[(size_t)BS * i + z] = c[z];
#pragma unroll
            for (int s = 0; s < NSLOT; s++) {
                const bool h = (m >> s) & 1u;
                const double *a = row + (h ? __popc(m & ((1u << s) - 1u)) * B2 : 0);
                double x = c[0] * (h ? a[0] : 0.0);
#pragma unroll
                for (int z = 1; z < BS; z++) x = x + c[z] * (h ? a[BS * z] : 0.0);
                app[(size_t)s * N + i] = x;
            }
        }
    }
    if (bad) atomicOr(flag, bad);
}

__global__ void k_any_nonfinite(long long n, const double *__restrict__ v, int32_t *__restrict__ flag) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && !isfinite(v[i])) atomicOr(flag, IMP_NONFINITE);
}

// y = alpha A x + beta y on the slot layout.  Each row sums its blocks in
// ascending column order and each block's entries in ascending order.  The
// workgroups run in launch order (not remapped per XCD), so the whole chip
// reads each of the 63 coefficient arrays at one advancing front, and the
// coefficients, read once per launch, are loaded non-temporally (streamed
// past the caches).  Measured on the 2M-cell grid this reads 12 % faster than
// one contiguous row range per XCD.
__global__ void __launch_bounds__(kBlock) k_slot_spmv(int nx, int ny, int nz, const double *__restrict__ A,
                                                      double alpha, const double *__restrict__ x, double beta,
                                                      double *__restrict__ y) {
    int n = nx * ny * nz;
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    size_t N = (size_t)n;
    int nxy = nx * ny;
    int ix = i % nx, iy = (i / nx) % ny, iz = i / nxy;
    const int nb[7] = {iz > 0 ? i - nxy : -1, iy > 0 ? i - nx : -1, ix > 0 ? i - 1 : -1, i,
                       ix < nx - 1 ? i + 1 : -1, iy < ny - 1 ? i + nx : -1, iz < nz - 1 ? i + nxy : -1};
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int s = 0; s < NSLOT; s++) {
        int j = nb[s];
        if (j < 0) continue;
        const double *a = A + (size_t)s * 9 * N + i;
        double x0 = x[3 * (size_t)j], x1 = x[3 * (size_t)j + 1], x2 = x[3 * (size_t)j + 2];
        double e[9];
#pragma unroll
        for (int z = 0; z < 9; z++) e[z] = __builtin_nontemporal_load(a + z * N);
        s0 = s0 + e[0] * x0; s0 = s0 + e[1] * x1; s0 = s0 + e[2] * x2;
        s1 = s1 + e[3] * x0; s1 = s1 + e[4] * x1; s1 = s1 + e[5] * x2;
        s2 = s2 + e[6] * x0; s2 = s2 + e[7] * x1; s2 = s2 + e[8] * x2;
    }
    double *yi = y + 3 * (size_t)i;
    if (beta == 0.0) {
        yi[0] = alpha * s0 + 0.0; yi[1] = alpha * s1 + 0.0; yi[2] = alpha * s2 + 0.0;
    } else {
        yi[0] = alpha * s0 + beta * yi[0];
        yi[1] = alpha * s1 + beta * yi[1];
        yi[2] = alpha * s2 + beta * yi[2];
    }
}

// r = v - A (Pi_p dp): only column 0 of each block is needed.  The residual
// is formed in FP64; dp may be FP32 (mixed form) and r is stored as TO.
template <typename TD, typename TO>
__global__ void __launch_bounds__(kBlock) k_slot_col0_residual(int nx, int ny, int nz,
                                                               const double *__restrict__ A,
                                                               const double *__restrict__ v,
                                                               const TD *__restrict__ dp,
                                                               TO *__restrict__ r) {
    int n = nx * ny * nz;
    int i = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    size_t N = (size_t)n;
    int nxy = nx * ny;
    int ix = i % nx, iy = (i / nx) % ny, iz = i / nxy;
    const int nb[7] = {iz > 0 ? i - nxy : -1, iy > 0 ? i - nx : -1, ix > 0 ? i - 1 : -1, i,
                       ix < nx - 1 ? i + 1 : -1, iy < ny - 1 ? i + nx : -1, iz < nz - 1 ? i + nxy : -1};
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int s = 0; s < NSLOT; s++) {
        int j = nb[s];
        if (j < 0) continue;
        const double *a = A + (size_t)s * 9 * N + i;
        double p = (double)dp[j];
        s0 = s0 + a[0 * N] * p;
        s1 = s1 + a[3 * N] * p;
        s2 = s2 + a[6 * N] * p;
    }
    r[3 * (size_t)i] = (TO)(v[3 * (size_t)i] - s0);
    r[3 * (size_t)i + 1] = (TO)(v[3 * (size_t)i + 1] - s1);
    r[3 * (size_t)i + 2] = (TO)(v[3 * (size_t)i + 2] - s2);
}

// The same residual written in the F stage's slot order: component c of cell
// i goes to out[c * S + slot_of[i]].
// ---- BLAS-1 -------------------------------------------------------------------
__global__ void k_axpby(long long n, double a, const double *__restrict__ x, double b, double *__restrict__ y) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    y[i] = b == 0.0 ? a * x[i] : a * x[i] + b * y[i];
}

// w <- w / sqrt(nrm2[0]) unless that norm is <= 1e-300 (Arnoldi breakdown):
// the same product (1/h) w as axpby with the factor formed on the host
__global__ void k_normalize(long long n, const double *__restrict__ nrm2, double *__restrict__ w) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double h = sqrt(nrm2[0]);
    if (h > 1e-300) w[i] = (1.0 / h) * w[i];
}

__global__ void k_fill(long long n, double v, double *__restrict__ y) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = v;
}

// x of the lane whose number differs in bit MASK (8, 4, 2 or 1): row moves
// within 16 lanes where the instruction has the pattern, LDS permutes for 4
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
    static_assert(MASK == 8 || MASK == 4 || MASK == 2 || MASK == 1, "within 16 lanes");
    if constexpr (MASK == 4) return (uint32_t)__shfl_xor((int)x, 4, 64);
    // row_ror:8, quad_perm [2,3,0,1], quad_perm [1,0,3,2]
    constexpr int ctrl = MASK == 8 ? 0x128 : MASK == 2 ? 0x4E : 0xB1;
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xF, 0xF, true);
}
// One step of a wavefront's butterfly sum over C values at once: lanes whose
// bit MASK is clear go on with the even values, the others with the odd ones,
// so a step halves the values and every value is added in the same order as a
// butterfly of its own, x[lane] + x[lane ^ MASK].  An odd value stays in both.
template <int MASK, int C>
__device__ __forceinline__ void fold(const double (&v)[C], double (&o)[(C + 1) / 2]) {
    auto lo = [](double x) { return (uint32_t)__double2loint(x); };
    auto hi = [](double x) { return (uint32_t)__double2hiint(x); };
    auto dbl = [](uint32_t l, uint32_t h) { return __hiloint2double((int)h, (int)l); };
#pragma unroll
    for (int i = 0; i < (C + 1) / 2; i++) {
        const double a = v[2 * i], b = v[2 * i + 1 < C ? 2 * i + 1 : 2 * i];
        if constexpr (MASK >= 16) {
            // the swap leaves [a, b] of the clear lanes in one register and
            // [a, b] of the set lanes in the other
            auto l = MASK == 32 ? __builtin_amdgcn_permlane32_swap(lo(a), lo(b), false, false)
                                : __builtin_amdgcn_permlane16_swap(lo(a), lo(b), false, false);
            auto h = MASK == 32 ? __builtin_amdgcn_permlane32_swap(hi(a), hi(b), false, false)
                                : __builtin_amdgcn_permlane16_swap(hi(a), hi(b), false, false);
            o[i] = dbl(l[0], h[0]) + dbl(l[1], h[1]);
        } else {
            const bool set = (threadIdx.x & MASK) != 0;
            const double keep = set ? b : a, send = set ? a : b;
            o[i] = keep + dbl(lane_xor<MASK>(lo(send)), lane_xor<MASK>(hi(send)));
        }
    }
}
// Wavefront sums of M values (M <= 64) in the order of a butterfly over lane
// distances 32, 16, ... 1: lane sum_index<M>() ends with one of the sums.  For
// M = 56 that is 56 exchanges of a double, where M butterflies take 336.
template <int M>
__device__ __forceinline__ double wave_sums(const double (&v)[M]) {
    constexpr int c1 = (M + 1) / 2, c2 = (c1 + 1) / 2, c3 = (c2 + 1) / 2, c4 = (c3 + 1) / 2, c5 = (c4 + 1) / 2;
    static_assert((c5 + 1) / 2 == 1, "at most 64 values");
    double o1[c1], o2[c2], o3[c3], o4[c4], o5[c5], o6[1];
    fold<32>(v, o1);
    fold<16>(o1, o2);
    fold<8>(o2, o3);
    fold<4>(o3, o4);
    fold<2>(o4, o5);
    fold<1>(o5, o6);
    return o6[0];
}
// which of the M sums this lane holds after wave_sums
template <int M>
__device__ __forceinline__ int sum_index() {
    constexpr int c1 = (M + 1) / 2, c2 = (c1 + 1) / 2, c3 = (c2 + 1) / 2, c4 = (c3 + 1) / 2, c5 = (c4 + 1) / 2;
    const int lane = threadIdx.x % 64;
    int q = 0;
    auto up = [&](int bit, int count) { q = min(2 * q + ((lane & bit) ? 1 : 0), count - 1); };
    up(1, c5);
    up(2, c4);
    up(4, c3);
    up(8, c2);
    up(16, c1);
    up(32, M);
    return q;
}
// Sums of M values over the workgroup: thread q < M returns the q-th, its
// wavefronts added in order.  sh may be used again after a barrier.
template <int M>
__device__ __forceinline__ double block_sums(const double (&v)[M], double (&sh)[M][kBlock / 64]) {
    const double t = wave_sums(v);
    sh[sum_index<M>()][threadIdx.x / 64] = t;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x < M) {
#pragma unroll
        for (int u = 0; u < kBlock / 64; u++) s = s + sh[threadIdx.x][u];
    }
    return s;
}

// The workgroups' part of a reduction of M sums: partial[q * blocks + block].
// With done set (a zeroed word) the workgroup that finishes last adds the
// partial sums as k_partial_final does, in the same order, and writes out (and
// mirror, pinned host memory): a launch less.  The partial sums are written
// through and read past the caches, so no fence writes back a whole L2; the
// word is zero again at the end.
template <int M>
__device__ __forceinline__ void finish_sums(const double (&acc)[M], double (&sh)[M][kBlock / 64], double *partial,
                                            uint32_t *done, double *out, double *mirror) {
    const double t = block_sums(acc, sh);
    const uint32_t nb = gridDim.x;
    if (!done) {
        if (threadIdx.x < M) partial[(size_t)threadIdx.x * nb + blockIdx.x] = t;
        return;
    }
    static_assert(M <= 64, "wavefront 0 holds the sums");
    __shared__ uint32_t ticket;
    if (threadIdx.x < 64) {
        if (threadIdx.x < M)
            __hip_atomic_store(&partial[(size_t)threadIdx.x * nb + blockIdx.x], t, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        stores_done();
        if (threadIdx.x == 0)
            ticket = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (ticket != nb - 1) return;
    double s[M];
#pragma unroll
    for (int q = 0; q < M; q++) s[q] = 0.0;
    for (uint32_t b = threadIdx.x; b < nb; b += kBlock) {
#pragma unroll
        for (int q = 0; q < M; q++)
            s[q] = s[q] + __hip_atomic_load(&partial[(size_t)q * nb + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const double r = block_sums(s, sh);
    if (threadIdx.x < M) {
        out[threadIdx.x] = r;
        if (mirror) mirror[threadIdx.x] = r;
    }
    if (threadIdx.x == 0) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Multi-dot, pass 1: each of the kRedBlocks workgroups writes the partial
// sums of its grid-stride share, partial[q * nblocks + block] = sum x[e] V[q][e].
template <int NV>
__global__ void __launch_bounds__(kBlock) k_multidot_partial(long long n, const double *__restrict__ x, VecList V,
                                                             double *__restrict__ partial, uint32_t *done,
                                                             double *out) {
    __shared__ double sh[NV][kBlock / 64];
    double acc[NV];
#pragma unroll
    for (int q = 0; q < NV; q++) acc[q] = 0.0;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        double xe = x[e];
#pragma unroll
        for (int q = 0; q < NV; q++) acc[q] = acc[q] + xe * V.p[q][e];
    }
    finish_sums(acc, sh, partial, done, out, nullptr);
}

// Classical Gram-Schmidt pass over the basis V (nv <= NV vectors), one read of
// every vector per element:
//   h == NULL:            partial sums of <w, V[q]>
//   h != NULL, dots != 0: w -= sum_q h[q] V[q], then partial sums of <w, V[q]>
//   h != NULL, dots == 0: w -= sum_q h[q] V[q], then the partial sum of <w, w>
// The basis values of an element stay in registers between the update and
// the dot products.  This form takes up to NV vectors (loads predicated on
// nv) and any length; k_cgs_exact below is the one the solver normally runs.
template <int NV>
__global__ void __launch_bounds__(kBlock) k_cgs_pass(long long n, double *__restrict__ w, VecList V, int nv,
                                                     const double *__restrict__ h, int dots,
                                                     double *__restrict__ partial) {
    __shared__ double hs[NV];
    __shared__ double sh[NV][kBlock / 64];
    if (h && threadIdx.x < nv) hs[threadIdx.x] = h[threadIdx.x];
    __syncthreads();
    double acc[NV];
#pragma unroll
    for (int q = 0; q < NV; q++) acc[q] = 0.0;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        double we = w[e];
        double vq[NV];
#pragma unroll
        for (int q = 0; q < NV; q++) vq[q] = q < nv ? V.p[q][e] : 0.0;
        if (h) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < NV; q++)
                if (q < nv) s = s + hs[q] * vq[q];
            we = we - s;
            w[e] = we;
        }
        if (dots || !h) {
#pragma unroll
            for (int q = 0; q < NV; q++) acc[q] = acc[q] + we * vq[q];
        } else {
            acc[0] = acc[0] + we * we;
        }
    }
    const double t = block_sums(acc, sh);
    if (threadIdx.x < ((dots || !h) ? nv : 1)) partial[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
}

// The same pass for exactly NV vectors below 4 GiB each, one kernel per mode
// (0: dots, 1: update then dots, 2: update then norm): no predicated loads (a
// load that only some paths issue makes the compiler wait for every load in
// flight) and no branches in the loop; each load is a vector base in scalar
// registers plus one 32-bit byte offset shared by all vectors, so addresses
// cost no vector registers.  Same arithmetic order as k_cgs_pass.
template <int NV, int MODE>
__global__ void __launch_bounds__(kBlock) k_cgs_exact(uint32_t n, double *__restrict__ w, VecList V,
                                                      const double *__restrict__ h, int rev,
                                                      double *__restrict__ partial, uint32_t *done, double *out) {
    constexpr bool upd = MODE != 0;
    constexpr int NA = MODE == 2 ? 1 : NV;  // accumulators
    __shared__ double hs[NV];
    __shared__ double sh[NA][kBlock / 64];
    if (upd && threadIdx.x < NV) hs[threadIdx.x] = h[threadIdx.x];
    __syncthreads();
    auto at = [](const double *p, uint32_t boff) -> const double * {
        return (const double *)((const char *)p + boff);
    };
    double acc[NA];
#pragma unroll
    for (int q = 0; q < NA; q++) acc[q] = 0.0;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        const uint32_t boff = (rev ? n - 1 - e : e) * (uint32_t)sizeof(double);
        double we = *at(w, boff);
        double vq[NV];
#pragma unroll
        for (int q = 0; q < NV; q++) vq[q] = *at(V.p[q], boff);
        if constexpr (upd) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < NV; q++) s = s + hs[q] * vq[q];
            we = we - s;
            *(double *)at(w, boff) = we;
        }
        if constexpr (MODE == 2) {
            acc[0] = acc[0] + we * we;
        } else {
#pragma unroll
            for (int q = 0; q < NV; q++) acc[q] = acc[q] + we * vq[q];
        }
    }
    finish_sums(acc, sh, partial, done, out, nullptr);
}

// ---- Gram-Schmidt with the re-orthogonalisation delayed by one step ---------
// (classical Gram-Schmidt twice, each vector's second projection taken in the
// step after it was formed, so one step reads the basis twice, not three
// times; Arnoldi step j has the final basis V[0..j), the pending vector
// V[j] = u (w of the previous step after its first projection) and w = A z_j)
//
// Dots: against u and w, for every vector of [V[0..j), u] (NV = j + 1):
// partial sums of <V[q], u> into rows q, of <V[q], w> into rows NV + q.
//
// Bound by the read of the NV + 1 vectors.  The compiler is told that two
// wavefronts per SIMD are enough: left to itself it keeps registers for eight
// and issues the loads of an element a few at a time; with all NV + 1 in
// flight, eight wavefronts per compute unit cover the latency.  The 2 NV sums
// of a wavefront are folded together (wave_sums): as butterflies of their own
// they took as long as the loads at 150 k elements.  Time with its final sums,
// before and now: 150 k elements, 8 vectors 13.7 and 6.4 us, 28 vectors 36.2
// and 8.8 us; 734 k, 20 vectors 48.1 and 23.1 us; 6 M, 12 vectors 162 and
// 104 us, 28 vectors 370 and 226 us (6.1 TB/s).  Up to three vectors are too few
// loads for eight wavefronts (48 M, one vector: 136 us, and 208 with two per SIMD).
template <int NV>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, NV < 4 ? 8 : 2)))
k_dcgs_dots(uint32_t n, VecList V, const double *__restrict__ w, double *__restrict__ partial, uint32_t *done,
            double *out, double *mirror) {
    __shared__ double sh[2 * NV][kBlock / 64];
    auto at = [](const double *p, uint32_t boff) -> const double * {
        return (const double *)((const char *)p + boff);
    };
    double acc[2 * NV];
#pragma unroll
    for (int q = 0; q < 2 * NV; q++) acc[q] = 0.0;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        const uint32_t boff = e * (uint32_t)sizeof(double);
        double we = *at(w, boff);
        double vq[NV];
#pragma unroll
        for (int q = 0; q < NV; q++) vq[q] = *at(V.p[q], boff);
        const double u = vq[NV - 1];
#pragma unroll
        for (int q = 0; q < NV; q++) {
            acc[q] = acc[q] + vq[q] * u;
            acc[NV + q] = acc[NV + q] + vq[q] * we;
        }
    }
    finish_sums(acc, sh, partial, done, out, mirror);
}

// Update for step J, from the dots red = [<V[i],u> (s_i), <u,u>, <V[i],w> (p_i),
// <u,w>]: beta = sqrt(<u,u> - |s|^2) (the norm of u - V s), the final vector
// v = (u - V s) / beta into V[J], r = <v,w> = (<u,w> - s.p) / beta, and
// w - V p - r v into V[J+1] (the next pending vector) with partial sums of
// its squared norm.  beta and r go to sc[0], sc[1] (workgroup 0); every
// workgroup forms the same coefficients.  A pending vector inside the span of
// the basis (beta^2 <= 0) leaves beta = 0 in sc[0] and zero vectors.
//
// Registers for two wavefronts per SIMD as in the dots, but not where they do not
// pay.  6 M elements with the compiler's choice and with two: step 11 149 and
// 125 us, step 27 353 and 275 us (5.4 TB/s), but step 15 160 and 173 us, step 19
// 197 and 211 us; 48 M: step 0 262 and 326 us, step 4 586 and 565 us.
template <int J>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, J < 2 || (J > 11 && J < 20) ? 8 : 2)))
k_dcgs_update(uint32_t n, VecList V, const double *__restrict__ red, double *__restrict__ sc, int rev,
              double *__restrict__ partial, double *sc_mirror, uint32_t *done, double *norm2, double *norm2_mirror) {
    __shared__ double cs[J > 0 ? J : 1], cp[J > 0 ? J : 1], cb[2];
    __shared__ double sh[1][kBlock / 64];
    if (threadIdx.x == 0) {
        double ss = 0.0, sp = 0.0;
        for (int i = 0; i < J; i++) {
            ss = ss + red[i] * red[i];
            sp = sp + red[i] * red[J + 1 + i];
        }
        double b2 = red[J] - ss, beta = 0.0, r = 0.0, ib = 0.0;
        if (b2 > 0.0) {
            beta = sqrt(b2);
            ib = 1.0 / beta;
            r = (red[2 * J + 1] - sp) / beta;
        }
        cb[0] = ib;
        cb[1] = r;
        if (blockIdx.x == 0) {
            sc[0] = beta; sc[1] = r;
            if (sc_mirror) { sc_mirror[0] = beta; sc_mirror[1] = r; }
        }
    }
    if (threadIdx.x < J) {
        cs[threadIdx.x] = red[threadIdx.x];
        cp[threadIdx.x] = red[J + 1 + threadIdx.x];
    }
    __syncthreads();
    const double ib = cb[0], r = ib > 0.0 ? cb[1] : 0.0;
    auto at = [](const double *p, uint32_t boff) -> double * {
        return (double *)((const char *)p + boff);
    };
    double acc[1] = {0.0};
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        const uint32_t boff = (rev ? n - 1 - e : e) * (uint32_t)sizeof(double);
        double vq[J > 0 ? J : 1];
#pragma unroll
        for (int q = 0; q < J; q++) vq[q] = *at(V.p[q], boff);
        double u = *at(V.p[J], boff), we = *at(V.p[J + 1], boff);
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int q = 0; q < J; q++) {
            s1 = s1 + cs[q] * vq[q];
            s2 = s2 + cp[q] * vq[q];
        }
        double v = (u - s1) * ib;
        double wn = we - s2 - r * v;
        *at(V.p[J], boff) = v;
        *at(V.p[J + 1], boff) = wn;
        acc[0] = acc[0] + wn * wn;
    }
    finish_sums(acc, sh, partial, done, norm2, norm2_mirror);
}

// pass 2 (one workgroup per result): out[q] = sum over the partials in a
// fixed order (strided per thread, then across the wavefront, then across the
// four wavefronts in order)
// (with mirror set, each result is also written there: pinned host memory
// the host reads after the stream's next event, instead of a copy)
__global__ void __launch_bounds__(kBlock) k_partial_final(int nblocks, const double *__restrict__ partial,
                                                          double *__restrict__ out, double *mirror = nullptr) {
    __shared__ double sh[1][kBlock / 64];
    const int q = blockIdx.x;
    double s[1] = {0.0};
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) s[0] = s[0] + partial[(size_t)q * nblocks + b];
    const double t = block_sums(s, sh);
    if (threadIdx.x == 0) {
        out[q] = t;
        if (mirror) mirror[q] = t;
    }
}

// y = y + sign * sum_q h[q] * V[q]  (h on the device)
__global__ void __launch_bounds__(kBlock) k_multiaxpy(long long n, VecList V, int nv,
                                                      const double *__restrict__ h, double sign,
                                                      double *__restrict__ y) {
    __shared__ double hs[kMaxVecList];
    if (threadIdx.x < nv) hs[threadIdx.x] = sign * h[threadIdx.x];
    __syncthreads();
    long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        double s = 0.0;
        for (int q = 0; q < nv; q++) s = s + hs[q] * V.p[q][e];
        y[e] = y[e] + s;
    }
}

__global__ void k_scale_copy(long long n, const double *__restrict__ inv, const double *__restrict__ x,
                             double *__restrict__ y) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = x[i] * inv[0];
}

// ---- host wrappers -------------------------------------------------------------
bo_status slot_spmv(const Grid &g, const double *A, double alpha, const double *x, double beta, double *y,
                    hipStream_t s) {
    long long n = g.n();
    k_slot_spmv<<<grid_for(n), kBlock, 0, s>>>(g.nx, g.ny, g.nz, A, alpha, x, beta, y);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

template <typename TD, typename TO>
bo_status slot_col0_residual(const Grid &g, const double *A, const double *v, const TD *dp, TO *r, hipStream_t s) {
    long long n = g.n();
    k_slot_col0_residual<TD, TO><<<grid_for(n), kBlock, 0, s>>>(g.nx, g.ny, g.nz, A, v, dp, r);
    BO_HIP(hipGetLastError());
    return BO_OK;
}
template bo_status slot_col0_residual<double, double>(const Grid &, const double *, const double *, const double *,
                                                      double *, hipStream_t);
template bo_status slot_col0_residual<float, double>(const Grid &, const double *, const double *, const float *,
                                                     double *, hipStream_t);

bo_status sell_build(int n, const int32_t *rp, const int32_t *ci, const double *v, const SellGrid &G,
                     DBuf<int32_t> &soff, DBuf<int32_t> &sci, DBuf<double> &sv, hipStream_t s) {
    int nsl = (n + 63) / 64;
    BO_TRY(soff.alloc((size_t)nsl + 1));
    int32_t *width = nullptr;
    BO_TRY(scratch_get(SC_SELL, sizeof(int32_t) * (size_t)std::max(nsl, 1), (void **)&width));
    k_sell_width<<<grid_for(64LL * nsl), kBlock, 0, s>>>(n, rp, ci, G, width);
    BO_HIP(hipGetLastError());
    int32_t cols = 0;
    BO_TRY(scan_counts(width, soff.p, nsl, &cols, s));
    BO_TRY(sci.alloc((size_t)cols * 64));
    BO_TRY(sv.alloc((size_t)cols * 64 * 9));
    if (n > 0) k_sell_fill<<<grid_for(n), kBlock, 0, s>>>(n, rp, ci, v, soff.p, G, sci.p, sv.p);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status sell_spmv(int n, const int32_t *soff, const int32_t *sci, const double *sv, const SellGrid &G,
                    double alpha, const double *x, double beta, double *y, hipStream_t s, const double *yin) {
    if (n <= 0) return BO_OK;
    k_sell_spmv<<<grid_for(n), kBlock, 0, s>>>(n, soff, sci, sv, G, alpha, x, beta, yin ? yin : y, y);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

template <typename TD>
bo_status sell_col0_update(int n, int npr, const int32_t *soff, const int32_t *sci, const double *sv,
                           const SellGrid &G, const TD *dp, double *r, hipStream_t s) {
    if (n <= 0) return BO_OK;
    k_sell_col0_update<TD><<<grid_for(n), kBlock, 0, s>>>(n, npr, soff, sci, sv, G, dp, r);
    BO_HIP(hipGetLastError());
    return BO_OK;
}
template bo_status sell_col0_update<double>(int, int, const int32_t *, const int32_t *, const double *,
                                            const SellGrid &, const double *, double *, hipStream_t);
template bo_status sell_col0_update<float>(int, int, const int32_t *, const int32_t *, const double *,
                                           const SellGrid &, const float *, double *, hipStream_t);

template <typename TD>
bo_status slot_col0_update(const Grid &g, const double *A, const TD *dp, double *r, hipStream_t s) {
    k_slot_col0_update<TD><<<grid_for(g.n()), kBlock, 0, s>>>(g.nx, g.ny, g.nz, A, dp, r);
    BO_HIP(hipGetLastError());
    return BO_OK;
}
template bo_status slot_col0_update<double>(const Grid &, const double *, const double *, double *, hipStream_t);
template bo_status slot_col0_update<float>(const Grid &, const double *, const float *, double *, hipStream_t);

template <int BS>
bo_status grid_import(const Grid &g, const int32_t *rp, const int32_t *ci, const double *v, long long nnzb, int mode,
                      double *slots, double *cw, double *app, int32_t *flag, const char *who, hipStream_t s) {
    const unsigned nb = grid_for(g.n(), kBsrRows);
    BO_HIP(hipMemsetAsync(flag, 0, sizeof(int32_t), s));
    if ((uintptr_t)v % 16 == 0)
        k_grid_import<BS, true><<<nb, 256, 0, s>>>(g.nx, g.ny, g.nz, rp, ci, v, mode, slots, cw, app, flag);
    else
        k_grid_import<BS, false><<<nb, 256, 0, s>>>(g.nx, g.ny, g.nz, rp, ci, v, mode, slots, cw, app, flag);
    BO_HIP(hipGetLastError());
    int32_t h = 0;
    HostRead r{flag, sizeof h, &h};
    BO_TRY(host_reads(&r, 1, s));
    if (((h & IMP_PATTERN) || nnzb != stencil_entries(g)) && !(h & IMP_NONFINITE)) {
        // a wrong pattern, or blocks behind the last row, leave values unread: a
        // value that is not finite comes first
        const long long nv = (long long)BS * BS * nnzb;
        k_any_nonfinite<<<grid_for(nv), kBlock, 0, s>>>(nv, v, flag);
        BO_HIP(hipGetLastError());
        BO_TRY(host_reads(&r, 1, s));
    }
    if (h & IMP_NONFINITE) return fail(BO_ERR_NONFINITE, std::string(who) + ": the matrix holds NaN or Inf");
    if (h & IMP_PATTERN)
        return fail(BO_ERR_UNSUPPORTED, std::string(who) + ": the pattern is not the grid's 7-point stencil");
    if (h & IMP_SINGULAR)
        return fail(BO_ERR_SINGULAR_BLOCK,
                    std::string(who) + ": singular saturation block (no quasi-IMPES decoupling)");
    return BO_OK;
}
template bo_status grid_import<2>(const Grid &, const int32_t *, const int32_t *, const double *, long long, int,
                                  double *, double *, double *, int32_t *, const char *, hipStream_t);
template bo_status grid_import<3>(const Grid &, const int32_t *, const int32_t *, const double *, long long, int,
                                  double *, double *, double *, int32_t *, const char *, hipStream_t);

bo_status axpby(long long n, double a, const double *x, double b, double *y, hipStream_t s) {
    k_axpby<<<grid_for(n), kBlock, 0, s>>>(n, a, x, b, y);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status normalize(long long n, const double *nrm2, double *w, hipStream_t s) {
    k_normalize<<<grid_for(n), kBlock, 0, s>>>(n, nrm2, w);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status fill(long long n, double v, double *y, hipStream_t s) {
    k_fill<<<grid_for(n), kBlock, 0, s>>>(n, v, y);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status multiaxpy(long long n, const double *const *Vhost, int nv, const double *h, double sign, double *y,
                    hipStream_t s) {
    if (nv > kMaxVecList || nv < 1) return fail(BO_ERR_INVALID_ARG, "multiaxpy: 1..64 vectors");
    VecList L{};
    for (int q = 0; q < nv; q++) L.p[q] = Vhost[q];
    long long blocks = std::min<long long>((n + kBlock - 1) / kBlock, 4096);
    k_multiaxpy<<<(unsigned)std::max<long long>(blocks, 1), kBlock, 0, s>>>(n, L, nv, h, sign, y);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status scale_copy(long long n, const double *inv, const double *x, double *y, hipStream_t s) {
    k_scale_copy<<<grid_for(n), kBlock, 0, s>>>(n, inv, x, y);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

__global__ void k_clear_word(uint32_t *w) { *w = 0; }

bo_status Reducer::init(hipStream_t s) {
    BO_TRY(partial.alloc((size_t)kRedBlocks * kMaxVecList));
    if (!done.p) {
        BO_TRY(done.alloc(1));
        k_clear_word<<<1, 1, 0, s>>>(done.p);
        BO_HIP(hipGetLastError());
    }
    return BO_OK;
}

// Workgroups of the Gram-Schmidt kernels: as many as are resident at once, at
// most four per compute unit (kRedBlocks on a full device), found once per
// kernel and device; a fixed count per kernel keeps the partial sums' order
// fixed.  Slots: k_cgs_exact<K, M> 4K + M, k_dcgs_dots<K> 4K + 3,
// k_dcgs_update<K> 4(kCgsExactMax + 1) + K.
constexpr int kCgsExactMax = 32;
static int resident_blocks(const void *kernel, int slot) {
    constexpr int kSlots = (kCgsExactMax + 1) * 5, kDevs = 16;
    static int cache[kDevs][kSlots] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevs) return kRedBlocks;
    int &c = cache[dev][slot];
    if (c == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 ||
            cus < 1)
            c = kRedBlocks;
        else
            c = std::min(kRedBlocks, std::min(per_cu, 4) * cus);
    }
    return c;
}

// Workgroups that a pass over n elements needs: one without an element would
// add a zero to the partial sums, in the order of the rest.
static int used_blocks(int nb, long long n) {
    return (int)std::max<long long>(1, std::min<long long>(nb, (n + kBlock - 1) / kBlock));
}

// Whether the workgroup that ends last adds up the partial sums itself instead
// of a second kernel: with few workgroups (up to 32 k elements).  Their counts
// go to one word one after the other, about 9 ns each.  Dots of 4 vectors with
// their final sums: in place 3.8 us at 6 k elements (24 workgroups) and 11.2
// at 150 k (586), where those by a second kernel take 6.1 us.
static bool finish_in_place(int nb) { return nb <= 128; }

bo_status Reducer::cgs_pass(long long n, double *w, const double *const *Vhost, int nv, const double *h, bool dots,
                            double *out, hipStream_t s, bool reverse) {
    if (nv < 1 || nv > kMaxVecList) return fail(BO_ERR_INVALID_ARG, "cgs_pass: 1..64 vectors");
    VecList L{};
    for (int q = 0; q < nv; q++) L.p[q] = Vhost[q];
    // a fixed grid per vector count (the partial sums' order does not depend
    // on the device), small enough to be resident at once
    int nb = kRedBlocks;
    const int nout = (dots || !h) ? nv : 1;
    bool fin = false;
    if (nv <= kCgsExactMax && n < (1ll << 29)) {
        const uint32_t n32 = (uint32_t)n;
        const int mode = !h ? 0 : dots ? 1 : 2, rev = reverse ? 1 : 0;
        switch (nv * 4 + mode) {
#define BO_CGS1(K, M)                                                                  \
    case K * 4 + M:                                                                    \
        nb = used_blocks(resident_blocks((const void *)k_cgs_exact<K, M>, K * 4 + M), n); \
        fin = finish_in_place(nb);                                               \
        k_cgs_exact<K, M><<<nb, kBlock, 0, s>>>(n32, w, L, h, rev, partial.p, fin ? done.p : nullptr, out); \
        break;
#define BO_CGS(K) BO_CGS1(K, 0) BO_CGS1(K, 1) BO_CGS1(K, 2)
            BO_CGS(1) BO_CGS(2) BO_CGS(3) BO_CGS(4) BO_CGS(5) BO_CGS(6) BO_CGS(7) BO_CGS(8)
            BO_CGS(9) BO_CGS(10) BO_CGS(11) BO_CGS(12) BO_CGS(13) BO_CGS(14) BO_CGS(15) BO_CGS(16)
            BO_CGS(17) BO_CGS(18) BO_CGS(19) BO_CGS(20) BO_CGS(21) BO_CGS(22) BO_CGS(23) BO_CGS(24)
            BO_CGS(25) BO_CGS(26) BO_CGS(27) BO_CGS(28) BO_CGS(29) BO_CGS(30) BO_CGS(31) BO_CGS(32)
#undef BO_CGS
#undef BO_CGS1
        default: break;
        }
    } else if (nv <= 8) {
        k_cgs_pass<8><<<nb, kBlock, 0, s>>>(n, w, L, nv, h, dots ? 1 : 0, partial.p);
    } else if (nv <= 16) {
        k_cgs_pass<16><<<nb, kBlock, 0, s>>>(n, w, L, nv, h, dots ? 1 : 0, partial.p);
    } else if (nv <= 32) {
        k_cgs_pass<32><<<nb, kBlock, 0, s>>>(n, w, L, nv, h, dots ? 1 : 0, partial.p);
    } else {
        k_cgs_pass<64><<<nb, kBlock, 0, s>>>(n, w, L, nv, h, dots ? 1 : 0, partial.p);
    }
    if (!fin) k_partial_final<<<nout, kBlock, 0, s>>>(nb, partial.p, out);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status Reducer::multidot_16(long long n, const double *x, const VecList &L, int nv, double *out, hipStream_t s) {
    const int nb = used_blocks(kRedBlocks, n);
    const bool fin = finish_in_place(nb);
    uint32_t *d = fin ? done.p : nullptr;
    switch (nv) {
#define BO_MD(K) case K: k_multidot_partial<K><<<nb, kBlock, 0, s>>>(n, x, L, partial.p, d, out); break;
        BO_MD(1) BO_MD(2) BO_MD(3) BO_MD(4) BO_MD(5) BO_MD(6) BO_MD(7) BO_MD(8)
        BO_MD(9) BO_MD(10) BO_MD(11) BO_MD(12) BO_MD(13) BO_MD(14) BO_MD(15) BO_MD(16)
#undef BO_MD
    default: break;
    }
    if (!fin) k_partial_final<<<nv, kBlock, 0, s>>>(nb, partial.p, out);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status Reducer::multidot(long long n, const double *x, const double *const *Vhost, int nv, double *out,
                            hipStream_t s) {
    for (int q0 = 0; q0 < nv; q0 += 16) {
        int c = std::min(16, nv - q0);
        VecList L{};
        for (int q = 0; q < c; q++) L.p[q] = Vhost[q0 + q];
        BO_TRY(multidot_16(n, x, L, c, out + q0, s));
    }
    return BO_OK;
}

bo_status Reducer::dcgs_dots(long long n, const double *const *Vhost, int nv, const double *w, double *out,
                             hipStream_t s, double *mirror) {
    if (nv < 1 || nv > kCgsExactMax || n >= (1ll << 29))
        return fail(BO_ERR_INVALID_ARG, "dcgs_dots: 1..32 vectors below 2^29 elements");
    VecList L{};
    for (int q = 0; q < nv; q++) L.p[q] = Vhost[q];
    const uint32_t n32 = (uint32_t)n;
    int nb = kRedBlocks;
    bool fin = false;
    switch (nv) {
#define BO_D(K)                                                                   \
    case K:                                                                       \
        nb = used_blocks(resident_blocks((const void *)k_dcgs_dots<K>, 4 * K + 3), n); \
        fin = finish_in_place(nb);                                         \
        k_dcgs_dots<K><<<nb, kBlock, 0, s>>>(n32, L, w, partial.p, fin ? done.p : nullptr, out, mirror); \
        break;
        BO_D(1) BO_D(2) BO_D(3) BO_D(4) BO_D(5) BO_D(6) BO_D(7) BO_D(8)
        BO_D(9) BO_D(10) BO_D(11) BO_D(12) BO_D(13) BO_D(14) BO_D(15) BO_D(16)
        BO_D(17) BO_D(18) BO_D(19) BO_D(20) BO_D(21) BO_D(22) BO_D(23) BO_D(24)
        BO_D(25) BO_D(26) BO_D(27) BO_D(28) BO_D(29) BO_D(30) BO_D(31) BO_D(32)
#undef BO_D
    default: break;
    }
    if (!fin) k_partial_final<<<2 * nv, kBlock, 0, s>>>(nb, partial.p, out, mirror);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status Reducer::dcgs_update(long long n, const double *const *Vhost, int j, const double *red, double *sc,
                               double *norm2, hipStream_t s, bool reverse, double *sc_mirror, double *norm2_mirror) {
    if (j < 0 || j + 1 > kCgsExactMax || n >= (1ll << 29))
        return fail(BO_ERR_INVALID_ARG, "dcgs_update: step 0..31 below 2^29 elements");
    VecList L{};
    for (int q = 0; q < j + 2; q++) L.p[q] = Vhost[q];
    const uint32_t n32 = (uint32_t)n;
    const int rev = reverse ? 1 : 0;
    int nb = kRedBlocks;
    bool fin = false;
    switch (j) {
#define BO_U(K)                                                                     \
    case K:                                                                         \
        nb = used_blocks(resident_blocks((const void *)k_dcgs_update<K>, 4 * (kCgsExactMax + 1) + K), n); \
        fin = finish_in_place(nb);                                                  \
        k_dcgs_update<K><<<nb, kBlock, 0, s>>>(n32, L, red, sc, rev, partial.p, sc_mirror, fin ? done.p : nullptr, \
                                               norm2, norm2_mirror);                \
        break;
        BO_U(0) BO_U(1) BO_U(2) BO_U(3) BO_U(4) BO_U(5) BO_U(6) BO_U(7)
        BO_U(8) BO_U(9) BO_U(10) BO_U(11) BO_U(12) BO_U(13) BO_U(14) BO_U(15)
        BO_U(16) BO_U(17) BO_U(18) BO_U(19) BO_U(20) BO_U(21) BO_U(22) BO_U(23)
        BO_U(24) BO_U(25) BO_U(26) BO_U(27) BO_U(28) BO_U(29) BO_U(30) BO_U(31)
#undef BO_U
    default: break;
    }
    if (!fin) k_partial_final<<<1, kBlock, 0, s>>>(nb, partial.p, norm2, norm2_mirror);
    BO_HIP(hipGetLastError());
    return BO_OK;
}

bo_status Reducer::dot(long long n, const double *x, const double *y, double *out, hipStream_t s) {
    VecList L{};
    L.p[0] = y;
    return multidot_16(n, x, L, 1, out, s);
}

}  // namespace bo

using namespace bo;

extern "C" const char *bo_last_error(void) { return g_err.c_str(); }
extern "C" const char *bo_version(void) { return "bo 0.1 (gfx950)"; }

extern "C" bo_status bo_bsr_spmv(const bo_bsr *A, double alpha, const double *x, double beta, double *y,
                                 void *stream) {
    if (!A || !x || !y || !A->rowptr || !A->colind || !A->val || A->nbrows < 0)
        return fail(BO_ERR_INVALID_ARG, "bo_bsr_spmv: NULL argument");
    if (A->nbrows == 0) return BO_OK;
    return bsr_spmv_launch<3>(A->nbrows, A->nnzb, A->rowptr, A->colind, A->val, alpha, x, beta, y,
                              (hipStream_t)stream);
}
