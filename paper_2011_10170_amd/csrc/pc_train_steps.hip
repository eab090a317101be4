// Training-side steps around the convolution path: pattern pool generation (Section 4.2), adaptive
// finalisation counters (Section 4.3) and the gradient of the modified group-lasso penalty (Section 4.4,
// Eq. 3 and Eq. 4). All are one pass over [F][C][9] float32 tensors: bound by HBM traffic.
//
// Results that are integers (masks, counts, picks) come from float32 arithmetic in a fixed order without
// fused multiply-add (this file is compiled with -ffp-contract=off) and from integer atomics only.
#include "pc_importance.h"

#include <algorithm>

#define TS_BLOCK 256

// 9 floats of TS_BLOCK consecutive kernels from global memory to LDS with contiguous loads.
__device__ __forceinline__ void ts_stage(float *dst, const float *__restrict__ src, int n)
{
    // all loads first (index clamped, so they are unconditional), then the LDS writes: one memory round trip
    float r[9];
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int i = j * TS_BLOCK + threadIdx.x;
        r[j] = src[i < n * 9 ? i : n * 9 - 1];
    }
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int i = j * TS_BLOCK + threadIdx.x;
        if (i < n * 9) dst[i] = r[j];
    }
}

// ------------------------------------------------------------------ pool generation, steps 1-4
// Tables by position, copied to LDS by every workgroup: n8[t] = neighbours of t as a bit mask, diagonals included (step 2);
// cand[9 * t1 + t2] = the candidates of step 3 (neighbours of t1 or t2 without diagonals, less the two themselves) in
// ascending order, four bits each, 15 = none. Two adjacent positions have 3 to 5 candidates.
struct TsDppgTable { uint32_t cand[81]; uint32_t n8[9]; };
constexpr bool ts_adjacent(int t, int u, bool diagonal)
{
    const int dr = u / 3 - t / 3, ds = u % 3 - t % 3, ar = dr < 0 ? -dr : dr, as = ds < 0 ? -ds : ds;
    return u != t && ar <= 1 && as <= 1 && (diagonal || ar + as == 1);
}
constexpr TsDppgTable ts_dppg_table()
{
    TsDppgTable r = {};
    for (int t = 0; t < 9; ++t)
        for (int u = 0; u < 9; ++u) {
            if (ts_adjacent(t, u, true)) r.n8[t] |= 1u << u;
            uint32_t w = 0xFFFFFu;
            int n = 0;
            for (int c = 0; c < 9; ++c)
                if (c != t && c != u && (ts_adjacent(t, c, false) || ts_adjacent(u, c, false)) && n < 5) {
                    w = (w & ~(15u << (4 * n))) | ((uint32_t)c << (4 * n));
                    ++n;
                }
            r.cand[9 * t + u] = w;
        }
    return r;
}
__device__ const TsDppgTable ts_dppg_tab = ts_dppg_table();

// Candidate pattern of every kernel of a chunk of n <= 64, counted in the LDS histogram lh; own: the thread's importances
// in LDS. Bound by vector instructions (1.63 M kernels 71 us while the neighbour sets were computed per kernel and all 36
// pairs of positions tried with 9 additions each): neighbour sets come from a table, and only the at most 10 pairs of the
// at most 5 candidates are tried.
__device__ __forceinline__ void ts_dppg_kernels(int n, int64_t k0, uint32_t *lh, const TsDppgTable &tab, uint16_t *__restrict__ masks,
                                                const float *own)
{
    const int lane = threadIdx.x & 63;
    if (lane < n) {
        float s[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) s[t] = own[t];
        // step 1: first maximum over the 9 positions (every update below is a select: no divergent branches)
        int t1 = 0;
        float b1 = s[0];
#pragma unroll
        for (int t = 1; t < 9; ++t) {
            const bool up = s[t] > b1;
            b1 = up ? s[t] : b1;
            t1 = up ? t : t1;
        }
        // step 2: first maximum over the neighbours of t1, diagonals included
        const uint32_t n8 = tab.n8[t1];
        int t2 = -1;
        float b2 = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const bool up = (((n8 >> t) & 1u) != 0u) & ((t2 < 0) | (s[t] > b2));
            b2 = up ? s[t] : b2;
            t2 = up ? t : t2;
        }
        // step 3: candidate positions and their importances
        const uint32_t cand = tab.cand[9 * t1 + t2];
        int c[5];
        float v[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            c[i] = (int)((cand >> (4 * i)) & 15u);
            v[i] = own[c[i] < 9 ? c[i] : 0];
            if (i >= 3) v[i] = c[i] < 9 ? v[i] : -__builtin_inff();   // no candidate: never the larger sum
        }
        // step 4: best pair of candidates (pairs in lexicographic order, the first one always exists). A sum adds the four
        // importances in ascending order of the positions; the terms of the two first positions enter before, between or
        // behind the pair, as +0 where they do not belong (importances are squares, never below +0: +0 changes no bit).
        const bool first_lo = t1 < t2;
        const int lo = first_lo ? t1 : t2, hi = first_lo ? t2 : t1;
        const float slo = first_lo ? b1 : b2, shi = first_lo ? b2 : b1;
        float hl[5], hh[5], tl[5], th[5], head[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            hl[i] = lo < c[i] ? slo : 0.0f;
            hh[i] = hi < c[i] ? shi : 0.0f;
            tl[i] = lo < c[i] ? 0.0f : slo;
            th[i] = hi < c[i] ? 0.0f : shi;
            head[i] = (hl[i] + hh[i]) + v[i];
        }
        float best = 0.0f;
        int best_ij = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = i + 1; j < 5; ++j) {
                const float ml = lo < c[i] ? 0.0f : hl[j], mh = hi < c[i] ? 0.0f : hh[j];
                const float acc = ((((head[i] + ml) + mh) + v[j]) + tl[j]) + th[j];
                const bool take = (i == 0 && j == 1) || acc > best;
                best = take ? acc : best;
                best_ij = take ? 4 * i + (4 * j << 8) : best_ij;
            }
        const uint32_t best_m = (1u << t1) | (1u << t2) | (1u << ((cand >> (best_ij & 255)) & 15u)) | (1u << ((cand >> (best_ij >> 8)) & 15u));
        atomicAdd(&lh[best_m], 1u);
        if (masks) masks[k0 + lane] = (uint16_t)best_m;
    }
}

// The layers of a network in one launch: chunk ch belongs to the layer l with blk0[l] <= ch < blk0[l + 1].
struct TsBatchArg {
    int32_t n;
    int32_t blk0[PC_BATCH_MAX + 1];
    int64_t nk[PC_BATCH_MAX];
    const float *W[PC_BATCH_MAX], *G[PC_BATCH_MAX];
    const uint8_t *pid[PC_BATCH_MAX], *keep[PC_BATCH_MAX];
    void *out[PC_BATCH_MAX];          // masks (pool generation), counts, picked ids or dW, by kernel
    const uint32_t *counts[PC_BATCH_MAX];
};

// Every wavefront takes units of 64 kernels (a quarter of a chunk of TS_BLOCK), the next unit on its way from memory while
// one is worked on; units that do not divide evenly go to different workgroups. Counts go to LDS and from there to the pool
// once, at the end: every workgroup adds to the same 44 live counters one behind the other, so there are few and large ones
// (1.63 M kernels: 47 us with 1597 workgroups of 256 threads).
#define TS_DPPG_BLOCK 1024
__global__ void __launch_bounds__(TS_DPPG_BLOCK) pc_dppg_batch_kernel(TsBatchArg b, uint32_t *__restrict__ hist)
{
    __shared__ __align__(16) float s[TS_DPPG_BLOCK / 64][64 * 9];
    __shared__ uint32_t lh[512];
    __shared__ TsDppgTable tab;
    if (threadIdx.x < 512) lh[threadIdx.x] = 0u;
    if (threadIdx.x < sizeof(TsDppgTable) / 4)
        reinterpret_cast<uint32_t *>(&tab)[threadIdx.x] = reinterpret_cast<const uint32_t *>(&ts_dppg_tab)[threadIdx.x];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    struct Unit { int l, n; int64_t k0; };
    int layer = 0;                              // units are walked in ascending order
    auto unit_of = [&](int64_t u) -> Unit {     // n <= 0: past the end of its layer
        const int ch = (int)(u >> 2);
        while (layer + 1 < b.n && ch >= b.blk0[layer + 1]) ++layer;
        Unit c;
        c.l = layer;
        c.k0 = (int64_t)(ch - b.blk0[layer]) * TS_BLOCK + (int)(u & 3) * 64;
        const int64_t left = b.nk[layer] - c.k0;
        c.n = left < 64 ? (int)left : 64;
        return c;
    };
    const int64_t total = 4 * (int64_t)b.blk0[b.n], step = (int64_t)gridDim.x * (TS_DPPG_BLOCK / 64);
    int64_t u = (int64_t)wave * gridDim.x + blockIdx.x;
    PcImpRegs r;
    Unit c = {0, 0, 0};
    if (u < total) c = unit_of(u);
    if (c.n > 0) pc_imp_issue(b.W[c.l], b.G[c.l], c.k0, c.n, r);
    while (u < total) {
        if (c.n > 0) pc_imp_put(r, b.G[c.l] != nullptr, c.n, s[wave]);
        const Unit now = c;
        u += step;
        if (u < total) {
            c = unit_of(u);
            if (c.n > 0) pc_imp_issue(b.W[c.l], b.G[c.l], c.k0, c.n, r);
        }
        ts_dppg_kernels(now.n, now.k0, lh, tab, static_cast<uint16_t *>(b.out[now.l]), s[wave] + (threadIdx.x & 63) * 9);
    }
    __syncthreads();
    if (threadIdx.x < 512 && lh[threadIdx.x]) atomicAdd(&hist[threadIdx.x], lh[threadIdx.x]);   // integer counts: the order of the additions does not matter
}

// Workgroups for n chunks of TS_BLOCK kernels: two fill a CU.
static unsigned ts_dppg_grid(const pc_ctx *ctx, int64_t n)
{
    const int64_t wgs = (n * (TS_BLOCK / 64) + TS_DPPG_BLOCK / 64 - 1) / (TS_DPPG_BLOCK / 64), most = 2 * (int64_t)ctx->num_cu;
    return (unsigned)(wgs < most ? wgs : most);
}

extern "C" pc_status pc_dppg_accumulate(pc_ctx *ctx, const float *W, const float *G, int32_t F, int32_t C,
                                        uint32_t *hist, uint16_t *masks)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    if (!W || !hist) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_dppg_accumulate: null pointer");
    if (F < 1 || C < 1 || F > 65535 || C > 65535)
        return pc_fail(ctx, PC_ERR_BAD_SHAPE, "pc_dppg_accumulate: F=%d C=%d out of range", F, C);
    PC_HIP(ctx, hipSetDevice(ctx->device));
    TsBatchArg b;
    memset(&b, 0, sizeof(b));
    b.n = 1;
    b.nk[0] = (int64_t)F * C;
    b.blk0[1] = (int32_t)((b.nk[0] + TS_BLOCK - 1) / TS_BLOCK);
    b.W[0] = W; b.G[0] = G; b.out[0] = masks;
    hipLaunchKernelGGL(pc_dppg_batch_kernel, dim3(ts_dppg_grid(ctx, b.blk0[1])), dim3(TS_DPPG_BLOCK), 0, ctx->stream, b, hist);
    return pc_hip_check(ctx, hipGetLastError(), "pool generation launch");
}

extern "C" pc_status pc_dppg_pool(pc_ctx *ctx, const uint32_t *hist, int32_t n_patterns, uint16_t *lib_host,
                                  uint32_t *score_host, int32_t *n_found)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    if (!hist || !lib_host || !n_found) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_dppg_pool: null pointer");
    if (n_patterns < 1 || n_patterns > PC_MAX_P)
        return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_dppg_pool: n_patterns=%d outside 1..%d", n_patterns, PC_MAX_P);
    PC_HIP(ctx, hipSetDevice(ctx->device));
    uint32_t h[512] = {};
    PC_HIP(ctx, hipMemcpyAsync(h, hist, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    PC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    int order[512], found = 0;
    for (int m = 0; m < 512; ++m)
        if (h[m]) order[found++] = m;
    std::sort(order, order + found, [&](int a, int b) { return h[a] != h[b] ? h[a] > h[b] : a < b; });   // (allocates nothing)
    const int n = found < n_patterns ? found : n_patterns;
    for (int i = 0; i < n; ++i) {
        lib_host[i] = (uint16_t)order[i];
        if (score_host) score_host[i] = h[order[i]];
    }
    *n_found = n;
    return PC_OK;
}

// ------------------------------------------------------------------ adaptive finalisation
__global__ void __launch_bounds__(256)
pc_finalize_count_kernel(const uint8_t *__restrict__ pid, int64_t nk, int P, uint32_t *__restrict__ counts)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nk) return;
    const int p = pid[k];
    if (p < P) counts[k * P + p] += 1u;             // one thread per kernel: no other thread touches this row
}

// First maximum of a kernel's P counters; 16-byte loads where the rows allow them, all of up to 16 counters at once.
__device__ __forceinline__ uint8_t ts_pick(const uint32_t *__restrict__ row, int P)
{
    int best = 0, p = 0;
    uint32_t bc = row[0];
    if ((P & 3) == 0 && (reinterpret_cast<uintptr_t>(row) & 15) == 0) {
        for (; p < P; p += 16) {
            uint4 q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = *reinterpret_cast<const uint4 *>(row + (p + 4 * j < P ? p + 4 * j : 0));   // counter 0 again is never larger
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t c[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (p + 4 * j < P && c[e] > bc) { bc = c[e]; best = p + 4 * j + e; }
            }
        }
    } else {
        for (p = 1; p < P; ++p) {
            const uint32_t c = row[p];
            if (c > bc) { bc = c; best = p; }
        }
    }
    return (uint8_t)best;
}

__global__ void __launch_bounds__(256)
pc_finalize_pick_kernel(const uint32_t *__restrict__ counts, int64_t nk, int P, uint8_t *__restrict__ pid)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nk) pid[k] = ts_pick(counts + k * P, P);
}

// One kernel per thread: what moves is a 64-byte line of counters per kernel in and out, at 5.5 TB/s (four kernels per
// thread: 45 us instead of 38 for 1.63 M kernels; the layer found by one vector load instead of a few scalar ones: 41).
__global__ void __launch_bounds__(256) pc_finalize_count_batch_kernel(TsBatchArg b, int P)
{
    int l = 0;
    while (l + 1 < b.n && (int)blockIdx.x >= b.blk0[l + 1]) ++l;
    const int64_t k = (int64_t)((int)blockIdx.x - b.blk0[l]) * 256 + threadIdx.x;
    if (k >= b.nk[l]) return;
    const int p = b.pid[l][k];
    if (p < P) static_cast<uint32_t *>(b.out[l])[k * P + p] += 1u;
}

__global__ void __launch_bounds__(256) pc_finalize_pick_batch_kernel(TsBatchArg b, int P)
{
    const int l = pc_batch_find(b.blk0, b.n, (int)blockIdx.x);
    const int64_t k = (int64_t)((int)blockIdx.x - b.blk0[l]) * 256 + threadIdx.x;
    if (k >= b.nk[l]) return;
    static_cast<uint8_t *>(b.out[l])[k] = ts_pick(b.counts[l] + k * P, P);
}

static pc_status ts_check_counts(pc_ctx *ctx, const char *who, const void *a, const void *b, int32_t F, int32_t C, int32_t P)
{
    if (!a || !b) return pc_fail(ctx, PC_ERR_INVALID_ARG, "%s: null pointer", who);
    if (F < 1 || C < 1 || F > 65535 || C > 65535) return pc_fail(ctx, PC_ERR_BAD_SHAPE, "%s: F=%d C=%d out of range", who, F, C);
    if (P < 1 || P > PC_MAX_P) return pc_fail(ctx, PC_ERR_BAD_LIBRARY, "%s: P=%d outside 1..%d", who, P, PC_MAX_P);
    return PC_OK;
}

extern "C" pc_status pc_finalize_count(pc_ctx *ctx, const uint8_t *pid, int32_t F, int32_t C, int32_t P, uint32_t *counts)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    pc_status s = ts_check_counts(ctx, "pc_finalize_count", pid, counts, F, C, P);
    if (s != PC_OK) return s;
    PC_HIP(ctx, hipSetDevice(ctx->device));
    const int64_t nk = (int64_t)F * C;
    hipLaunchKernelGGL(pc_finalize_count_kernel, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, ctx->stream, pid, nk, P, counts);
    return pc_hip_check(ctx, hipGetLastError(), "finalisation count launch");
}

extern "C" pc_status pc_finalize_pick(pc_ctx *ctx, const uint32_t *counts, int32_t F, int32_t C, int32_t P, uint8_t *pid)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    pc_status s = ts_check_counts(ctx, "pc_finalize_pick", counts, pid, F, C, P);
    if (s != PC_OK) return s;
    PC_HIP(ctx, hipSetDevice(ctx->device));
    const int64_t nk = (int64_t)F * C;
    hipLaunchKernelGGL(pc_finalize_pick_kernel, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, ctx->stream, counts, nk, P, pid);
    return pc_hip_check(ctx, hipGetLastError(), "finalisation pick launch");
}

// ------------------------------------------------------------------ modified group lasso
// One thread per kernel; W and dW pass through LDS so that global accesses are contiguous.
__device__ __forceinline__ void ts_group_lasso_block(const float *__restrict__ W, const uint8_t *__restrict__ pid,
                                                     const uint8_t *__restrict__ keep, int64_t nk, const LibArg &la, float lambda_p,
                                                     float lambda_i, float *__restrict__ dW, double *__restrict__ block_pen,
                                                     int blk)
{
    __shared__ float sw[TS_BLOCK * 9], sd[TS_BLOCK * 9];
    __shared__ uint16_t lmask[PC_MAX_P + 2];
    __shared__ double red[TS_BLOCK / 64];
    const int64_t k0 = (int64_t)blk * TS_BLOCK;
    const int n = nk - k0 < TS_BLOCK ? (int)(nk - k0) : TS_BLOCK;
    if (threadIdx.x < la.P) lmask[threadIdx.x] = la.mask[threadIdx.x];
    ts_stage(sw, W + k0 * 9, n);
    ts_stage(sd, dW + k0 * 9, n);
    int p = 0, kp = 1;
    if (threadIdx.x < n) { p = pid[k0 + threadIdx.x]; kp = keep[k0 + threadIdx.x]; }
    __syncthreads();
    double pen = 0.0;
    if (threadIdx.x < n) {
        const unsigned m = p < la.P ? lmask[p] : 0x1FFu;   // an id outside the pool penalises nothing by pattern
        float w[9];
        float zn2 = 0.0f, un2 = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            w[t] = sw[threadIdx.x * 9 + t];
            const float sq = w[t] * w[t];
            zn2 = zn2 + (((m >> t) & 1u) ? 0.0f : sq);
            un2 = un2 + sq;
        }
        if (kp) un2 = 0.0f;
        const float zn = sqrtf(zn2), un = sqrtf(un2);
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            float g = 0.0f;
            if (!((m >> t) & 1u) && zn > 0.0f) g = lambda_p * (w[t] / zn);
            if (!kp && un > 0.0f) g = g + lambda_i * (w[t] / un);
            sd[threadIdx.x * 9 + t] += g;
        }
        pen = (double)lambda_p * (double)zn + (double)lambda_i * (double)un;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int i = j * TS_BLOCK + threadIdx.x;
        if (i < n * 9) dW[k0 * 9 + i] = sd[i];
    }
    if (block_pen) {                                // fixed-order tree over the workgroup
        for (int d = 32; d > 0; d >>= 1) pen += __shfl_down(pen, d);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = pen;
        __syncthreads();
        if (threadIdx.x == 0) block_pen[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);    // one slot per workgroup of the launch
    }
}

__global__ void __launch_bounds__(TS_BLOCK)
pc_group_lasso_kernel(const float *__restrict__ W, const uint8_t *__restrict__ pid, const uint8_t *__restrict__ keep, int64_t nk,
                      LibArg la, float lambda_p, float lambda_i, float *__restrict__ dW, double *__restrict__ block_pen)
{
    ts_group_lasso_block(W, pid, keep, nk, la, lambda_p, lambda_i, dW, block_pen, (int)blockIdx.x);
}

__global__ void __launch_bounds__(TS_BLOCK)
pc_group_lasso_batch_kernel(TsBatchArg b, LibArg la, float lambda_p, float lambda_i, double *__restrict__ block_pen)
{
    const int l = pc_batch_find(b.blk0, b.n, (int)blockIdx.x);
    ts_group_lasso_block(b.W[l], b.pid[l], b.keep[l], b.nk[l], la, lambda_p, lambda_i, static_cast<float *>(b.out[l]), block_pen,
                         (int)blockIdx.x - b.blk0[l]);
}

// penalty = the workgroup sums added in a fixed order by one workgroup: a thread requests 8 of its values at a time
// (6385 sums: one memory round trip; with 256 threads adding one value behind the other 7.9 us)
__global__ void __launch_bounds__(1024) pc_group_lasso_sum_kernel(const double *__restrict__ block_pen, int nb, double *__restrict__ out)
{
    __shared__ double red[16];
    double s = 0.0;
    for (int i0 = 0; i0 < nb; i0 += 8192) {
        double v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = i0 + j * 1024 + (int)threadIdx.x;
            v[j] = block_pen[i < nb ? i : nb - 1];
            if (i >= nb) v[j] = 0.0;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < 16; ++w) t += red[w];
        *out = t;
    }
}

extern "C" pc_status pc_group_lasso_grad(pc_ctx *ctx, const float *W, const uint8_t *pid, const uint8_t *keep, int32_t F,
                                         int32_t C, const uint16_t *lib, int32_t P, float lambda_p, float lambda_i,
                                         float *dW, double *penalty)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    if (!W || !pid || !keep || !lib || !dW) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_group_lasso_grad: null pointer");
    if (F < 1 || C < 1 || F > 65535 || C > 65535)
        return pc_fail(ctx, PC_ERR_BAD_SHAPE, "pc_group_lasso_grad: F=%d C=%d out of range", F, C);
    pc_status s = pc_check_library(lib, P);
    if (s != PC_OK) return pc_fail(ctx, s, "pc_group_lasso_grad: bad library (P=%d)", P);
    PC_HIP(ctx, hipSetDevice(ctx->device));
    LibArg la;
    pc_fill_lib(&la, lib, P);
    const int64_t nk = (int64_t)F * C;
    const unsigned nb = (unsigned)((nk + TS_BLOCK - 1) / TS_BLOCK);
    double *block_pen = nullptr;
    if (penalty) {
        void *scr = nullptr;
        s = pc_scratch(ctx, sizeof(double) * nb, &scr);
        if (s != PC_OK) return s;
        block_pen = (double *)scr;
    }
    hipLaunchKernelGGL(pc_group_lasso_kernel, dim3(nb), dim3(TS_BLOCK), 0, ctx->stream, W, pid, keep, nk, la, lambda_p, lambda_i,
                       dW, block_pen);
    if (penalty)
        hipLaunchKernelGGL(pc_group_lasso_sum_kernel, dim3(1), dim3(1024), 0, ctx->stream, block_pen, (int)nb, penalty);
    return pc_hip_check(ctx, hipGetLastError(), "group lasso launch");
}

// ------------------------------------------------------------------ the same steps for the layers of a network at once
// Fills the table for layers [l0, l0 + m); false with a message when a layer is malformed.
static pc_status ts_fill_batch(pc_ctx *ctx, const char *who, TsBatchArg *b, int l0, int m, const int32_t *F, const int32_t *C)
{
    memset(b, 0, sizeof(*b));
    b->n = m;
    for (int i = 0; i < m; ++i) {
        const int l = l0 + i;
        if (F[l] < 1 || C[l] < 1 || F[l] > 65535 || C[l] > 65535)
            return pc_fail(ctx, PC_ERR_BAD_SHAPE, "%s: layer %d: F=%d C=%d out of range", who, l, F[l], C[l]);
        b->nk[i] = (int64_t)F[l] * C[l];
        b->blk0[i + 1] = b->blk0[i] + (int32_t)((b->nk[i] + TS_BLOCK - 1) / TS_BLOCK);
    }
    return PC_OK;
}

extern "C" pc_status pc_dppg_accumulate_batch(pc_ctx *ctx, int32_t n_layers, const float *const *W, const float *const *G,
                                              const int32_t *F, const int32_t *C, uint32_t *hist, uint16_t *const *masks)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    if (n_layers < 0) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_dppg_accumulate_batch: n_layers %d", n_layers);
    if (n_layers == 0) return PC_OK;
    if (!W || !F || !C || !hist) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_dppg_accumulate_batch: null pointer");
    for (int l = 0; l < n_layers; ++l)
        if (!W[l]) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_dppg_accumulate_batch: null pointer in layer %d", l);
    PC_HIP(ctx, hipSetDevice(ctx->device));
    for (int l0 = 0; l0 < n_layers; l0 += PC_BATCH_MAX) {
        const int m = n_layers - l0 < PC_BATCH_MAX ? n_layers - l0 : PC_BATCH_MAX;
        TsBatchArg b;
        pc_status s = ts_fill_batch(ctx, "pc_dppg_accumulate_batch", &b, l0, m, F, C);
        if (s != PC_OK) return s;
        for (int i = 0; i < m; ++i) {
            b.W[i] = W[l0 + i];
            b.G[i] = G ? G[l0 + i] : nullptr;
            b.out[i] = masks ? masks[l0 + i] : nullptr;
        }
        hipLaunchKernelGGL(pc_dppg_batch_kernel, dim3(ts_dppg_grid(ctx, b.blk0[m])), dim3(TS_DPPG_BLOCK), 0, ctx->stream, b, hist);
    }
    return pc_hip_check(ctx, hipGetLastError(), "pool generation (several layers) launch");
}

extern "C" pc_status pc_finalize_count_batch(pc_ctx *ctx, int32_t n_layers, const uint8_t *const *pid, const int32_t *F,
                                             const int32_t *C, int32_t P, uint32_t *const *counts)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    if (n_layers < 0) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_finalize_count_batch: n_layers %d", n_layers);
    if (n_layers == 0) return PC_OK;
    if (!pid || !F || !C || !counts) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_finalize_count_batch: null pointer");
    if (P < 1 || P > PC_MAX_P) return pc_fail(ctx, PC_ERR_BAD_LIBRARY, "pc_finalize_count_batch: P=%d outside 1..%d", P, PC_MAX_P);
    for (int l = 0; l < n_layers; ++l)
        if (!pid[l] || !counts[l]) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_finalize_count_batch: null pointer in layer %d", l);
    PC_HIP(ctx, hipSetDevice(ctx->device));
    for (int l0 = 0; l0 < n_layers; l0 += PC_BATCH_MAX) {
        const int m = n_layers - l0 < PC_BATCH_MAX ? n_layers - l0 : PC_BATCH_MAX;
        TsBatchArg b;
        pc_status s = ts_fill_batch(ctx, "pc_finalize_count_batch", &b, l0, m, F, C);
        if (s != PC_OK) return s;
        for (int i = 0; i < m; ++i) { b.pid[i] = pid[l0 + i]; b.out[i] = counts[l0 + i]; }
        hipLaunchKernelGGL(pc_finalize_count_batch_kernel, dim3((unsigned)b.blk0[m]), dim3(256), 0, ctx->stream, b, P);
    }
    return pc_hip_check(ctx, hipGetLastError(), "finalisation count (several layers) launch");
}

extern "C" pc_status pc_finalize_pick_batch(pc_ctx *ctx, int32_t n_layers, const uint32_t *const *counts, const int32_t *F,
                                            const int32_t *C, int32_t P, uint8_t *const *pid)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    if (n_layers < 0) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_finalize_pick_batch: n_layers %d", n_layers);
    if (n_layers == 0) return PC_OK;
    if (!pid || !F || !C || !counts) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_finalize_pick_batch: null pointer");
    if (P < 1 || P > PC_MAX_P) return pc_fail(ctx, PC_ERR_BAD_LIBRARY, "pc_finalize_pick_batch: P=%d outside 1..%d", P, PC_MAX_P);
    for (int l = 0; l < n_layers; ++l)
        if (!pid[l] || !counts[l]) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_finalize_pick_batch: null pointer in layer %d", l);
    PC_HIP(ctx, hipSetDevice(ctx->device));
    for (int l0 = 0; l0 < n_layers; l0 += PC_BATCH_MAX) {
        const int m = n_layers - l0 < PC_BATCH_MAX ? n_layers - l0 : PC_BATCH_MAX;
        TsBatchArg b;
        pc_status s = ts_fill_batch(ctx, "pc_finalize_pick_batch", &b, l0, m, F, C);
        if (s != PC_OK) return s;
        for (int i = 0; i < m; ++i) { b.counts[i] = counts[l0 + i]; b.out[i] = pid[l0 + i]; }
        hipLaunchKernelGGL(pc_finalize_pick_batch_kernel, dim3((unsigned)b.blk0[m]), dim3(256), 0, ctx->stream, b, P);
    }
    return pc_hip_check(ctx, hipGetLastError(), "finalisation pick (several layers) launch");
}

extern "C" pc_status pc_group_lasso_grad_batch(pc_ctx *ctx, int32_t n_layers, const float *const *W, const uint8_t *const *pid,
                                               const uint8_t *const *keep, const int32_t *F, const int32_t *C, const uint16_t *lib,
                                               int32_t P, float lambda_p, float lambda_i, float *const *dW, double *penalty)
{
    if (!ctx) return PC_ERR_INVALID_ARG;
    if (n_layers < 0) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_group_lasso_grad_batch: n_layers %d", n_layers);
    if (n_layers == 0) return PC_OK;
    if (!W || !pid || !keep || !F || !C || !lib || !dW) return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_group_lasso_grad_batch: null pointer");
    if (n_layers > PC_BATCH_MAX && penalty)
        return pc_fail(ctx, PC_ERR_UNSUPPORTED, "pc_group_lasso_grad_batch: the penalty of more than %d layers takes several calls", PC_BATCH_MAX);
    for (int l = 0; l < n_layers; ++l)
        if (!W[l] || !pid[l] || !keep[l] || !dW[l])
            return pc_fail(ctx, PC_ERR_INVALID_ARG, "pc_group_lasso_grad_batch: null pointer in layer %d", l);
    pc_status s = pc_check_library(lib, P);
    if (s != PC_OK) return pc_fail(ctx, s, "pc_group_lasso_grad_batch: bad library (P=%d)", P);
    PC_HIP(ctx, hipSetDevice(ctx->device));
    LibArg la;
    pc_fill_lib(&la, lib, P);
    for (int l0 = 0; l0 < n_layers; l0 += PC_BATCH_MAX) {
        const int m = n_layers - l0 < PC_BATCH_MAX ? n_layers - l0 : PC_BATCH_MAX;
        TsBatchArg b;
        s = ts_fill_batch(ctx, "pc_group_lasso_grad_batch", &b, l0, m, F, C);
        if (s != PC_OK) return s;
        for (int i = 0; i < m; ++i) {
            b.W[i] = W[l0 + i]; b.pid[i] = pid[l0 + i]; b.keep[i] = keep[l0 + i]; b.out[i] = dW[l0 + i];
        }
        const int nb = b.blk0[m];
        double *block_pen = nullptr;
        if (penalty) {
            void *scr = nullptr;
            s = pc_scratch(ctx, sizeof(double) * (size_t)nb, &scr);
            if (s != PC_OK) return s;
            block_pen = (double *)scr;
        }
        hipLaunchKernelGGL(pc_group_lasso_batch_kernel, dim3((unsigned)nb), dim3(TS_BLOCK), 0, ctx->stream, b, la, lambda_p, lambda_i,
                           block_pen);
        if (penalty)
            hipLaunchKernelGGL(pc_group_lasso_sum_kernel, dim3(1), dim3(1024), 0, ctx->stream, block_pen, nb, penalty);
    }
    return pc_hip_check(ctx, hipGetLastError(), "group lasso (several layers) launch");
}
