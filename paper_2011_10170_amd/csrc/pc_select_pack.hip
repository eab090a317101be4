// Pattern/kernel selection (Section 4.1, Eq. 1 and Eq. 2) and packing (Section 5.1) kernels.
//
// Selection is bit-reproducible: float32, fixed operation order, no fused multiply-add
// (this file must be compiled with -ffp-contract=off).
#include "pc_importance.h"
#include "pc_mfma.h"

// ------------------------------------------------------------------ selection
// Tap importances of one kernel -> best pattern of the pool and the ranking score. Every sum is taken in ascending tap
// order, one rounded float32 addition at a time. s points to the thread's 9 importances in LDS: the taps of a pattern are
// the same for the whole wavefront (scalar loads from the kernel arguments), so a pattern is 4 LDS reads and 3 additions.
// (With the importances in registers a pattern took 9 additions of s_t or +0, i.e. 9 bit tests and selects besides:
// selection of 1.63 M kernels with 16 patterns 48 us, bound by those vector instructions.)
__device__ __forceinline__ void pc_score_taps(const float *s, const LibArg &la, int score_mode, int *pid_out, float *rank_out)
{
    int best = 0;
    float best_score = 0.0f;
#pragma unroll 4
    for (int p = 0; p < la.P; ++p) {
        const uint32_t w = *reinterpret_cast<const uint32_t *>(la.taps[p]);
        const float acc = ((s[w & 255u] + s[(w >> 8) & 255u]) + s[(w >> 16) & 255u]) + s[w >> 24];
        if (p == 0 || acc > best_score) {
            best_score = acc;
            best = p;
        }
    }
    *pid_out = best;
    if (score_mode == PC_SCORE_KERNEL) {
        float acc = s[0];
#pragma unroll
        for (int t = 1; t < 9; ++t) acc = acc + s[t];
        *rank_out = acc;
    } else {
        *rank_out = best_score;
    }
}

// Scores of all kernels for the segments ranked by the kernels below; the first nzero words of zero are cleared for them.
__global__ void __launch_bounds__(256)
pc_select_score_kernel(const float *__restrict__ W, const float *__restrict__ G, int64_t nk, LibArg la, int score_mode,
                       uint8_t *__restrict__ pid, float *__restrict__ R, uint32_t *__restrict__ zero, int nzero)
{
    __shared__ __align__(16) float s[4][64 * 9];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = (int)blockIdx.x * 256 + (int)threadIdx.x; i < nzero; i += (int)gridDim.x * 256) zero[i] = 0u;
    const int64_t k0 = ((int64_t)blockIdx.x * 4 + wave) * 64;
    if (k0 >= nk) return;
    const int n = nk - k0 < 64 ? (int)(nk - k0) : 64;
    PcImpRegs r;
    pc_imp_issue(W, G, k0, n, r);
    pc_imp_put(r, G != nullptr, n, s[wave]);
    if (lane >= n) return;
    int best;
    float sc;
    pc_score_taps(s[wave] + lane * 9, la, score_mode, &best, &sc);
    pid[k0 + lane] = (uint8_t)best;
    R[k0 + lane] = sc;
}

// ---- exact top-n of a segment in the order (score descending, index ascending): a radix select over order-preserving
// 32-bit keys. A pass counts the next digit of the keys that share the prefix found so far; the digit that holds the
// rem-th largest of them joins the prefix. As soon as all keys of that digit are kept the rest of the key does not
// matter; otherwise, after the last digit, the keys equal to the threshold are kept by index. Counts are integers: the
// result does not depend on the order of the atomics.
#define PC_TOPN_WG 16384        // longest layer ranked by one workgroup (16384 kernels: 9.9 us; 16640 by the binned ranking 10.7)
__device__ __forceinline__ uint32_t pc_order_key(float f)
{
    const uint32_t b = __float_as_uint(f);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);   // a > b as floats  <=>  key(a) > key(b) as unsigned
}

// The digit of a finished histogram of T * PER bins (h: bins PER * threadIdx.x .. of this thread) that holds the rem-th
// largest key, 1 <= rem <= keys counted: in out[0], with the number of keys of larger digits in out[1] and its own count in
// out[2]. Called by all T threads; ends with a barrier. part: T / 64 ints of LDS.
template <int T, int PER>
__device__ __forceinline__ void pc_topn_digit(const uint32_t (&h)[PER], int rem, int *part, int *out)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) mine += (int)h[j];
    int incl = mine;                            // bins of this lane and of the higher lanes of the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_down(incl, off);
        if (lane + off < 64) incl += t;
    }
    if (lane == 0) part[wave] = incl;
    __syncthreads();
    int above = incl - mine;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) above += w > wave ? part[w] : 0;
    if (above < rem && rem <= above + mine) {   // exactly one thread
#pragma unroll
        for (int j = PER - 1; j >= 0; --j) {
            const int n = (int)h[j];
            if (above < rem && rem <= above + n) { out[0] = tid * PER + j; out[1] = above; out[2] = n; }
            above += n;
        }
    }
    __syncthreads();
}

// Position of each of the flagged elements among the flagged elements of the workgroup, by thread; *total: their number.
__device__ __forceinline__ int pc_block_rank(bool flag, int *wcnt, int nwaves, int *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long b = __ballot(flag);
    __syncthreads();                            // wcnt of an earlier call has been read
    if (lane == 0) wcnt[wave] = __popcll(b);
    __syncthreads();
    int before = __popcll(b & ((1ull << lane) - 1ull)), sum = 0;
    for (int w = 0; w < nwaves; ++w) {
        before += w < wave ? wcnt[w] : 0;
        sum += wcnt[w];
    }
    *total = sum;
    return before;
}

// A row's keys in one wavefront, key i in register i / 64 of lane i % 64 (registers past the row hold 0): keep flags of the
// registers j0 <= j < j1. The threshold comes from a binary search over the bits of the key: a step is one comparison per
// register, the lanes that pass are counted by the scalar unit, and no LDS or barrier takes part. It ends when exactly
// n_keep keys pass (after about 20 steps), or with the threshold key itself, whose copies are kept by index.
#define PC_ROW_MAX 512          // longest row ranked in registers
template <int NV>
__device__ __forceinline__ void pc_row_keep(const uint32_t (&key)[NV], int C, int n_keep, int j0, int j1, uint8_t *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    uint32_t T = 0u;
    int above = 0, cnt = -1;                    // keys known to exceed every later threshold; keys that pass T (-1: not counted)
    if (n_keep >= C) {
        cnt = n_keep;
    } else if (n_keep <= 0) {
        T = 0xFFFFFFFFu;
    } else {
        for (int bit = 31; bit >= 0 && cnt != n_keep; --bit) {
            const uint32_t t = T | (1u << bit);
            int c = 0;
#pragma unroll
            for (int j = 0; j < NV; ++j) c += (int)__popcll(__ballot(key[j] >= t));
            if (c >= n_keep) { T = t; cnt = c; }
            else above = c;
        }
    }
    const bool all = cnt == n_keep;             // every key that passes T is kept
    int rank = 0;                               // otherwise: keys equal to T seen so far, of which the first n_keep - above stay
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        bool take = key[j] >= T;
        if (!all) {
            const bool eq = key[j] == T && j * 64 + lane < C;
            const unsigned long long b = __ballot(eq);
            take = key[j] > T || (eq && rank + (int)__popcll(b & ((1ull << lane) - 1ull)) < n_keep - above);
            rank += (int)__popcll(b);
        }
        if (j >= j0 && j < j1 && j * 64 + lane < C) out[j * 64 + lane] = n_keep > 0 && take ? 1 : 0;
    }
}

// Selection of one filter row of at most 64 * NV kernels by one wavefront (s: 64 * 9 floats of LDS): the next 64 kernels
// are on their way from memory while 64 are scored.
template <int NV>
__device__ __forceinline__ void pc_select_row_wave(const float *__restrict__ W, const float *__restrict__ G, int C, const LibArg &la,
                                                   int score_mode, int n_keep, uint8_t *__restrict__ pid,
                                                   uint8_t *__restrict__ keep, int row, float *s)
{
    const int lane = threadIdx.x & 63;
    const int64_t row0 = (int64_t)row * C;
    uint32_t key[NV];
    PcImpRegs r;
    pc_imp_issue(W, G, row0, C < 64 ? C : 64, r);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        key[j] = 0u;
        const int n = C - j * 64 < 64 ? C - j * 64 : 64;
        if (n > 0) {
            pc_imp_put(r, G != nullptr, n, s);
            if (n == 64 && C > (j + 1) * 64)
                pc_imp_issue(W, G, row0 + (j + 1) * 64, C - (j + 1) * 64 < 64 ? C - (j + 1) * 64 : 64, r);
            if (lane < n) {
                int best;
                float sc;
                pc_score_taps(s + lane * 9, la, score_mode, &best, &sc);
                pid[row0 + j * 64 + lane] = (uint8_t)best;
                key[j] = pc_order_key(sc);
            }
        }
    }
    pc_row_keep<NV>(key, C, n_keep, 0, NV, keep + row0);
}

// One row of at most PC_ROW_MAX kernels per workgroup of ceil(C / 64) wavefronts, for launches with too few rows to fill the
// chip with a wavefront each: every wavefront scores 64 kernels, then all of them find the threshold of the whole row (one
// barrier, no second one) and each writes its own part.
__device__ __forceinline__ void pc_select_row_group(const float *__restrict__ W, const float *__restrict__ G, int C, const LibArg &la,
                                                    int score_mode, int n_keep, uint8_t *__restrict__ pid,
                                                    uint8_t *__restrict__ keep, int row)
{
    __shared__ __align__(16) float s[PC_ROW_MAX / 64][64 * 9];
    __shared__ uint32_t keys[PC_ROW_MAX];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)row * C;
    const int n = C - wave * 64 < 64 ? C - wave * 64 : 64;
    if (n > 0) {
        PcImpRegs r;
        pc_imp_issue(W, G, row0 + wave * 64, n, r);
        pc_imp_put(r, G != nullptr, n, s[wave]);
        if (lane < n) {
            int best;
            float sc;
            pc_score_taps(s[wave] + lane * 9, la, score_mode, &best, &sc);
            pid[row0 + wave * 64 + lane] = (uint8_t)best;
            keys[wave * 64 + lane] = pc_order_key(sc);
        }
    }
    __syncthreads();
    if (n <= 0) return;
    if (C <= 64) {
        const uint32_t key[1] = {lane < C ? keys[lane] : 0u};
        pc_row_keep<1>(key, C, n_keep, wave, wave + 1, keep + row0);
    } else {
        uint32_t key[PC_ROW_MAX / 64];
#pragma unroll
        for (int j = 0; j < PC_ROW_MAX / 64; ++j) key[j] = j * 64 + lane < C ? keys[j * 64 + lane] : 0u;
        pc_row_keep<PC_ROW_MAX / 64>(key, C, n_keep, wave, wave + 1, keep + row0);
    }
}

// Filter rows of several layers in one launch; PER_WAVE: a wavefront (workgroup of 64) per row, else a workgroup per row.
// Row b - row0[l] of the layer l whose range holds b.
struct SelBatchArg {
    int32_t n, score_mode;
    int32_t row0[PC_BATCH_MAX + 1];
    int32_t C[PC_BATCH_MAX], n_keep[PC_BATCH_MAX];
    const float *W[PC_BATCH_MAX], *G[PC_BATCH_MAX];
    uint8_t *pid[PC_BATCH_MAX], *keep[PC_BATCH_MAX];
};

template <bool PER_WAVE>
__global__ void __launch_bounds__(PER_WAVE ? 64 : PC_ROW_MAX) pc_select_rows_kernel(SelBatchArg b, LibArg la)
{
    const int l = pc_batch_find(b.row0, b.n, (int)blockIdx.x), row = (int)blockIdx.x - b.row0[l], C = b.C[l];
    if constexpr (PER_WAVE) {
        __shared__ __align__(16) float s[64 * 9];
        if (C <= 64) pc_select_row_wave<1>(b.W[l], b.G[l], C, la, b.score_mode, b.n_keep[l], b.pid[l], b.keep[l], row, s);
        else pc_select_row_wave<PC_ROW_MAX / 64>(b.W[l], b.G[l], C, la, b.score_mode, b.n_keep[l], b.pid[l], b.keep[l], row, s);
    } else {
        pc_select_row_group(b.W[l], b.G[l], C, la, b.score_mode, b.n_keep[l], b.pid[l], b.keep[l], row);
    }
}

// Top n_keep of segment blockIdx.x of R (L <= 1024 * NV scores): one workgroup with the keys in registers, digits of 12,
// 10 and 10 bits. A 256 x 256 layer ranked as a whole: one launch where counting across workgroups took eight (zeroing,
// four digits, equal scores, their scan, writing: 44 us with the gaps between them).
template <int NV>
__global__ void __launch_bounds__(1024)
pc_topn_wg_kernel(const float *__restrict__ R, int L, int n_keep, uint8_t *__restrict__ keep)
{
    __shared__ uint32_t hist[4096];
    __shared__ int part[16], dig[3];
    const float *seg = R + (int64_t)blockIdx.x * L;
    uint8_t *out = keep + (int64_t)blockIdx.x * L;
    const int tid = threadIdx.x;
    float r[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = j * 1024 + tid;
        r[j] = seg[i < L ? i : L - 1];
    }
    for (int i = tid; i < 4096; i += 1024) hist[i] = 0u;
    uint32_t prefix = 0u;
    int rem = n_keep, shift = 20;
    bool all;
    for (int pass = 0;; ++pass, shift -= 10) {
        const uint32_t himask = pass == 0 ? 0u : 0xFFFFFFFFu << (shift + 10);
        const uint32_t dmask = pass == 0 ? 4095u : 1023u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const uint32_t k = pc_order_key(r[j]);
            if (j * 1024 + tid < L && (k & himask) == prefix) atomicAdd(&hist[(k >> shift) & dmask], 1u);
        }
        __syncthreads();
        if (pass == 0) {
            const uint32_t h[4] = {hist[4 * tid], hist[4 * tid + 1], hist[4 * tid + 2], hist[4 * tid + 3]};
            pc_topn_digit<1024, 4>(h, rem, part, dig);
        } else {
            const uint32_t h[1] = {hist[tid]};
            pc_topn_digit<1024, 1>(h, rem, part, dig);
        }
        prefix |= (uint32_t)dig[0] << shift;
        rem -= dig[1];
        all = dig[2] == rem;
        if (all || shift == 0) break;
        hist[tid] = 0u;                         // read before the barrier that ended pc_topn_digit
    }
    const uint32_t himask = 0xFFFFFFFFu << shift;
    int base = 0;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = j * 1024 + tid;
        const uint32_t k = pc_order_key(r[j]);
        bool take = (k & himask) >= prefix;
        if (!all) {                             // uniform: of the keys equal to the threshold the first rem by index
            const bool eq = i < L && k == prefix;
            int total;
            const int before = base + pc_block_rank(eq, part, 16, &total);
            take = k > prefix || (eq && before < rem);
            base += total;
        }
        if (i < L) out[i] = take ? 1 : 0;
    }
}

// Rows of PC_ROW_MAX + 1 .. PC_ROW_LONG kernels of several layers in one launch, a workgroup per row: every wavefront scores 64
// kernels at a time, the keys stay in LDS (a thread ranks those it wrote) and the workgroup ranks them. No score goes through
// memory and the call needs no scratch. Bound by HBM where the rows fill the chip: 16 layers of 1024 x 1024 222 us = 5.6 TB/s,
// in two launches per layer with the scores in scratch 437 us (16 of 256 x 768: 45, 172 us). FEW, for at most one row per CU:
// bound by the scoring of a row on one CU, so more wavefronts, each with two units of 64 on their way (16 rows of 8192: 34 -> 26 us).
#define PC_ROW_LONG 8192        // longest row ranked in LDS
template <bool FEW>
__global__ void __launch_bounds__(FEW ? 1024 : 512) pc_select_long_rows_kernel(SelBatchArg b, LibArg la)
{
    constexpr int T = FEW ? 1024 : 512, DEPTH = FEW ? 2 : 1;   // threads; units of 64 kernels a wavefront has on their way
    extern __shared__ uint32_t keys[];          // as many as the longest row of the launch
    __shared__ __align__(16) float s[T / 64][64 * 9];   // staged importances, then the histogram
    __shared__ int part[T / 64], dig[3];
    static_assert(sizeof(s) >= 4096 * sizeof(uint32_t), "the histogram takes the place of the staged importances");
    const int l = pc_batch_find(b.row0, b.n, (int)blockIdx.x), row = (int)blockIdx.x - b.row0[l], C = b.C[l], n_keep = b.n_keep[l];
    const float *W = b.W[l], *G = b.G[l];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)row * C;
    uint8_t *out = b.keep[l] + row0;
    PcImpRegs r[DEPTH];
    auto issue = [&](int k, PcImpRegs &to) __attribute__((always_inline)) {
        if (k < C) pc_imp_issue(W, G, row0 + k, C - k < 64 ? C - k : 64, to);
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) issue(wave * 64 + d * T, r[d]);
    for (int k0 = wave * 64; k0 < C; k0 += DEPTH * T) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int k = k0 + d * T, n = C - k < 64 ? C - k : 64;
            if (n <= 0) break;
            pc_imp_put(r[d], G != nullptr, n, s[wave]);
            issue(k + DEPTH * T, r[d]);
            if (lane < n) {
                int best;
                float sc;
                pc_score_taps(s[wave] + lane * 9, la, b.score_mode, &best, &sc);
                b.pid[l][row0 + k + lane] = (uint8_t)best;
                keys[k + lane] = pc_order_key(sc);
            }
        }
    }
    const int tid = threadIdx.x;
    if (n_keep <= 0 || n_keep >= C) {
        for (int i = tid; i < C; i += T) out[i] = n_keep > 0 ? 1 : 0;
        return;
    }
    // as pc_topn_wg_kernel
    uint32_t *hist = reinterpret_cast<uint32_t *>(s);
    __syncthreads();                            // the staged importances have been read
    for (int i = tid; i < 4096; i += T) hist[i] = 0u;
    uint32_t prefix = 0u;
    int rem = n_keep, shift = 20;
    bool all;
    for (int pass = 0;; ++pass, shift -= 10) {
        const uint32_t himask = pass == 0 ? 0u : 0xFFFFFFFFu << (shift + 10);
        const uint32_t dmask = pass == 0 ? 4095u : 1023u;
        __syncthreads();
        for (int i = tid; i < C; i += T) {
            const uint32_t key = keys[i];
            if ((key & himask) == prefix) atomicAdd(&hist[(key >> shift) & dmask], 1u);
        }
        __syncthreads();
        if (pass == 0) {
            uint32_t h[4096 / T];
#pragma unroll
            for (int i = 0; i < 4096 / T; ++i) h[i] = hist[4096 / T * tid + i];
            pc_topn_digit<T, 4096 / T>(h, rem, part, dig);
        } else {
            uint32_t h[1024 / T];
#pragma unroll
            for (int i = 0; i < 1024 / T; ++i) h[i] = hist[1024 / T * tid + i];
            pc_topn_digit<T, 1024 / T>(h, rem, part, dig);
        }
        prefix |= (uint32_t)dig[0] << shift;
        rem -= dig[1];
        all = dig[2] == rem;
        if (all || shift == 0) break;
#pragma unroll
        for (int i = tid; i < 1024; i += T) hist[i] = 0u;   // read before the barrier that ended pc_topn_digit
    }
    const uint32_t himask = 0xFFFFFFFFu << shift;
    if (all) {
        for (int i = tid; i < C; i += T) out[i] = (keys[i] & himask) >= prefix ? 1 : 0;
        return;
    }
    int base = 0;                               // of the keys equal to the threshold the first rem by index
    for (int i0 = 0; i0 < C; i0 += T) {
        const int i = i0 + tid;
        const uint32_t key = i < C ? keys[i] : 0u;
        const bool eq = i < C && key == prefix;
        int total;
        const int before = base + pc_block_rank(eq, part, T / 64, &total);
        if (i < C) out[i] = key > prefix || (eq && before < rem) ? 1 : 0;
        base += total;
    }
}

// Segments above PC_TOPN_WG (whole layers ranked at once), across workgroups: three counting passes (11, 11 and 10 bits;
// hist[3][2048], zeroed by the score kernel) and a writing pass. Every workgroup walks its chunk of the scores and derives
// the prefix again from the finished histograms instead of reading it from a single writer; the last counting pass leaves
// the histogram of every chunk, from which the writing pass takes the number of threshold keys in the chunks before.
#define PC_TOPN_CHUNKS 1024     // at most so many chunks
#define PC_TOPN_BINS 2048
struct TopnState { uint32_t prefix; int rem, count; };   // count: keys that share the prefix

// UPTO finished passes; their histograms are requested together. The caller's next LDS use of part and dig needs no barrier.
template <int UPTO>
__device__ __forceinline__ TopnState pc_topn_replay(const uint32_t *__restrict__ hist, int n_keep, int *part, int *dig)
{
    TopnState s = {0u, n_keep, 0};
    uint32_t h[UPTO > 0 ? UPTO : 1][PC_TOPN_BINS / 256];
#pragma unroll
    for (int q = 0; q < UPTO; ++q) {
        const uint4 *src = reinterpret_cast<const uint4 *>(hist + q * PC_TOPN_BINS) + threadIdx.x * 2;
        const uint4 a = src[0], b = src[1];
        h[q][0] = a.x; h[q][1] = a.y; h[q][2] = a.z; h[q][3] = a.w;
        h[q][4] = b.x; h[q][5] = b.y; h[q][6] = b.z; h[q][7] = b.w;
    }
#pragma unroll
    for (int q = 0; q < UPTO; ++q) {
        pc_topn_digit<256, PC_TOPN_BINS / 256>(h[q], s.rem, part, dig);
        s.prefix |= (uint32_t)dig[0] << (q == 0 ? 21 : q == 1 ? 10 : 0);
        s.rem -= dig[1];
        s.count = dig[2];
        __syncthreads();
    }
    return s;
}

template <int PASS>
__global__ void __launch_bounds__(256)
pc_topn_hist_kernel(const float *__restrict__ R, int64_t L, int64_t chunk, int n_keep, uint32_t *__restrict__ hist,
                    uint32_t *__restrict__ chunk_hist)
{
    constexpr int SHIFT = PASS == 0 ? 21 : PASS == 1 ? 10 : 0, BINS = PASS == 2 ? 1024 : PC_TOPN_BINS;
    constexpr uint32_t HIMASK = PASS == 0 ? 0u : PASS == 1 ? 0xFFFFFFFFu << 21 : 0xFFFFFFFFu << 10;
    __shared__ uint32_t lh[BINS];
    __shared__ int part[4], dig[3];
    const int tid = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = i0 + chunk < L ? i0 + chunk : L;
    float r[4];                                 // the next 1024 scores, on their way during the replay
    auto load = [&](int64_t j0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = R[j0 + j * 256 + tid < i1 ? j0 + j * 256 + tid : i1 - 1];
    };
    load(i0);
    for (int i = tid; i < BINS; i += 256) lh[i] = 0u;
    const TopnState s = pc_topn_replay<PASS>(hist, n_keep, part, dig);
    __syncthreads();
    for (int64_t j0 = i0; j0 < i1; j0 += 1024) {
        uint32_t k[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) k[j] = pc_order_key(r[j]);
        if (j0 + 1024 < i1) load(j0 + 1024);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j0 + j * 256 + tid < i1 && (k[j] & HIMASK) == s.prefix) atomicAdd(&lh[(k[j] >> SHIFT) & (uint32_t)(BINS - 1)], 1u);
    }
    __syncthreads();
    for (int i = tid; i < BINS; i += 256) {
        const uint32_t c = lh[i];
        if (c) atomicAdd(&hist[PASS * PC_TOPN_BINS + i], c);   // integers: order-free
        if (PASS == 2) chunk_hist[(int64_t)blockIdx.x * 1024 + i] = c;
    }
}

// keep = 1 for scores above the threshold and for the first of the scores equal to it (by index).
__global__ void __launch_bounds__(256)
pc_topn_write_kernel(const float *__restrict__ R, int64_t L, int64_t chunk, int n_keep, const uint32_t *__restrict__ hist,
                     const uint32_t *__restrict__ chunk_hist, uint8_t *__restrict__ keep)
{
    __shared__ int part[4], dig[3], s_base;
    const int tid = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = i0 + chunk < L ? i0 + chunk : L;
    float r[4];
    auto load = [&](int64_t j0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = R[j0 + j * 256 + tid < i1 ? j0 + j * 256 + tid : i1 - 1];
    };
    load(i0);
    const TopnState s = pc_topn_replay<3>(hist, n_keep, part, dig);
    if (s.count == s.rem) {                     // all scores equal to the threshold are kept
        for (int64_t j0 = i0; j0 < i1; j0 += 1024) {
            uint8_t q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = pc_order_key(r[j]) >= s.prefix ? 1 : 0;
            if (j0 + 1024 < i1) load(j0 + 1024);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j0 + j * 256 + tid < i1) keep[j0 + j * 256 + tid] = q[j];
        }
        return;
    }
    if (tid == 0) s_base = 0;
    __syncthreads();
    int before_chunk = 0;
    for (int c = tid; c < (int)blockIdx.x; c += 256) before_chunk += (int)chunk_hist[(int64_t)c * 1024 + (s.prefix & 1023u)];
    if (before_chunk) atomicAdd(&s_base, before_chunk);
    __syncthreads();
    int base = s_base;
    for (int64_t j0 = i0; j0 < i1; j0 += 256) {
        const int64_t i = j0 + tid;
        const uint32_t k = i < i1 ? pc_order_key(R[i]) : 0u;
        const bool eq = i < i1 && k == s.prefix;
        int total;
        const int before = base + pc_block_rank(eq, part, 4, &total);
        if (i < i1) keep[i] = (k > s.prefix || (eq && before < s.rem)) ? 1 : 0;
        base += total;
    }
}

// Layers of PC_TOPN_WG + 1 .. PC_TOPN_BINNED kernels ranked as a whole, two launches. The scoring launch leaves, for every 1024 kernels
// ("row"), the keys grouped by bin (sign, exponent and first bit of the mantissa, largest first) and where each bin begins. A workgroup of
// the second launch adds up the rows' bin starts, which names the bin of the threshold, and walks that bin's keys of all rows, a tenth of
// the layer, itself; then it flags its own row. So nothing is handed from one workgroup to another but through the end of a launch, and no
// histogram has to be cleared. What bounds both is latency: the walk is a chain of bin starts, keys and two counting passes in LDS.
// Selection of 256 x 256 kernels: 17.3 us with the three counting launches and the writing one above, each waiting for the one before,
// 11.8 here; 130 x 128 16.3, 10.7. With more kernels the launches take little longer, while the walk grows with the rows and with the keys of the
// bin, most of them where half is kept. 10, 30 and 50 % kept, in a graph, launches / here: 73728 kernels 16.1, 16.5, 16.6 / 11.7, 14.0, 15.4; 82944 16.4, 16.9, 16.9 / 13.3, 14.9, 16.7;
// 92160 16.4, 17.0, 16.9 / 13.8, 16.8, 17.6; 102400 16.9, 17.3, 17.4 / 13.9, 16.2, 15.8: past the line every wavefront has a fifth row and
// half of the layer kept gains 1 us, then nothing.
#define PC_TOPN_BINNED 65536
#define PC_BIN_ROW 1024
#define PC_BINS 512
#define PC_BIN_PITCH 520        // starts of a row's bins: PC_BINS + 1, a multiple of 8
// Bin of a key, 0 for the largest: the upper 10 bits of positive scores; the last bin holds every other key too.
__device__ __forceinline__ int pc_key_bin(uint32_t key)
{
    const uint32_t top = key >> 22;
    return 1023 - (int)(top < 512u ? 512u : top);
}

__global__ void __launch_bounds__(PC_BIN_ROW)
pc_select_bins_kernel(const float *__restrict__ W, const float *__restrict__ G, int nk, LibArg la, int score_mode,
                      uint8_t *__restrict__ pid, uint32_t *__restrict__ R, uint32_t *__restrict__ K, uint16_t *__restrict__ start)
{
    __shared__ __align__(16) float s[16][64 * 9];
    __shared__ int cnt[PC_BINS], part[PC_BINS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row0 = (int)blockIdx.x * PC_BIN_ROW, k0 = row0 + wave * 64;
    const int n = nk - k0 < 64 ? nk - k0 : 64;  // kernels of this wavefront, none where negative
    PcImpRegs r;
    if (n > 0) pc_imp_issue(W, G, k0, n, r);
    if (tid < PC_BINS) cnt[tid] = 0;
    __syncthreads();
    uint32_t key = 0u;
    int rank = 0;
    if (n > 0) {
        pc_imp_put(r, G != nullptr, n, s[wave]);
        if (lane < n) {
            int best;
            float sc;
            pc_score_taps(s[wave] + lane * 9, la, score_mode, &best, &sc);
            key = pc_order_key(sc);
            pid[k0 + lane] = (uint8_t)best;
            R[k0 + lane] = key;
            rank = atomicAdd(&cnt[pc_key_bin(key)], 1);   // the order inside a bin does not matter: it is counted only
        }
    }
    __syncthreads();
    int incl = 0, mine = 0;
    if (tid < PC_BINS) {
        incl = mine = cnt[tid];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(incl, off);
            if (lane >= off) incl += t;
        }
        if (lane == 63) part[wave] = incl;
    }
    __syncthreads();
    if (tid < PC_BINS) {
        int first = incl - mine;
#pragma unroll
        for (int w = 0; w < PC_BINS / 64; ++w) first += w < wave ? part[w] : 0;
        cnt[tid] = first;
        uint16_t *to = start + (int64_t)blockIdx.x * PC_BIN_PITCH;
        to[tid] = (uint16_t)first;
        if (tid == PC_BINS - 1) to[PC_BINS] = (uint16_t)(first + mine);
    }
    __syncthreads();
    if (lane < n) K[row0 + cnt[pc_key_bin(key)] + rank] = key;
}

// The first 128 keys of a row's bin stay in registers; what follows is read in every pass.
__global__ void __launch_bounds__(PC_BIN_ROW)
pc_topn_bins_kernel(const uint32_t *__restrict__ R, const uint32_t *__restrict__ K, const uint16_t *__restrict__ start, int nk, int n_keep,
                    uint8_t *__restrict__ keep)
{
    constexpr int NR = PC_TOPN_BINNED / PC_BIN_ROW / 16;   // rows a wavefront walks, at most
    __shared__ int cum[PC_BINS + 1];            // keys of the layer in the bins before
    __shared__ uint32_t hist[2048];
    __shared__ int part[16], dig[3], s_bin, s_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = (int)gridDim.x, own = (int)blockIdx.x * PC_BIN_ROW + tid;
    const uint32_t mykey = R[own < nk ? own : nk - 1];
    if (tid <= PC_BINS) cum[tid] = 0;
    hist[tid] = 0u;
    hist[tid + 1024] = 0u;
    __syncthreads();
    {
        const int col = tid & 255;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(start) + col;
        int lo = 0, hi = 0;
#pragma unroll 8
        for (int r = tid >> 8; r < rows; r += 4) {
            const uint32_t u = src[r * (PC_BIN_PITCH / 2)];
            lo += (int)(u & 0xFFFFu);
            hi += (int)(u >> 16);
        }
        atomicAdd(&cum[2 * col], lo);           // integers: order-free
        atomicAdd(&cum[2 * col + 1], hi);
        if (tid == 0) cum[PC_BINS] = nk;
    }
    __syncthreads();
    if (tid < PC_BINS && cum[tid] < n_keep && n_keep <= cum[tid + 1]) s_bin = tid;   // exactly one thread: 0 < n_keep < nk
    __syncthreads();
    const int bin = s_bin, mybin = pc_key_bin(mykey);
    int rem = n_keep - cum[bin];
    if (rem == cum[bin + 1] - cum[bin]) {       // the whole bin is kept
        if (own < nk) keep[own] = mybin <= bin ? 1 : 0;
        return;
    }
    // the bin's keys of rows wave, wave + 16, ...: lane i holds the bounds of the i-th
    int b0 = 0, b1 = 0;
    if (lane < NR && wave + 16 * lane < rows) {
        const uint16_t *at = start + (wave + 16 * lane) * PC_BIN_PITCH + bin;
        b0 = at[0];
        b1 = at[1];
    }
    uint32_t q[NR][2];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int f = __builtin_amdgcn_readlane(b0, i), n = __builtin_amdgcn_readlane(b1, i) - f, row = wave + 16 * i < rows ? wave + 16 * i : 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) q[i][j] = K[row * PC_BIN_ROW + (j * 64 + lane < n ? f + j * 64 + lane : 0)];
    }
    auto walk = [&](auto &&use) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int f = __builtin_amdgcn_readlane(b0, i), n = __builtin_amdgcn_readlane(b1, i) - f;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (j * 64 + lane < n) use(q[i][j], i);
            for (int j = 128 + lane; j < n; j += 64) use(K[(wave + 16 * i) * PC_BIN_ROW + f + j], i);
        }
    };
    // digits of up to 11 bits of the keys of the bin: 22 bits are open, 32 in the last bin
    uint32_t prefix = bin == PC_BINS - 1 ? 0u : (uint32_t)(1023 - bin) << 22;
    int shift = bin == PC_BINS - 1 ? 32 : 22;
    bool all;
    for (;;) {
        const int width = shift < 11 ? shift : 11;
        const uint32_t himask = shift == 32 ? 0u : 0xFFFFFFFFu << shift;
        shift -= width;
        walk([&](uint32_t k, int) __attribute__((always_inline)) {
            if ((k & himask) == prefix) atomicAdd(&hist[(k >> shift) & ((1u << width) - 1u)], 1u);
        });
        __syncthreads();
        const uint32_t h[2] = {hist[2 * tid], hist[2 * tid + 1]};
        pc_topn_digit<1024, 2>(h, rem, part, dig);
        prefix |= (uint32_t)dig[0] << shift;
        rem -= dig[1];
        all = dig[2] == rem;
        if (all || shift == 0) break;
        hist[tid] = 0u;                         // read before the barrier that ended pc_topn_digit
        hist[tid + 1024] = 0u;
        __syncthreads();
    }
    if (all) {                                  // (keys below the bin are below its prefix, keys above it above)
        if (own < nk) keep[own] = (mykey & (0xFFFFFFFFu << shift)) >= prefix ? 1 : 0;
        return;
    }
    // of the keys equal to the threshold the first rem by index
    if (tid == 0) s_base = 0;
    __syncthreads();
    int before = 0;
    walk([&](uint32_t k, int i) __attribute__((always_inline)) { before += k == prefix && wave + 16 * i < (int)blockIdx.x; });
    if (before) atomicAdd(&s_base, before);
    const bool eq = own < nk && mykey == prefix;
    int total;
    const int rank = pc_block_rank(eq, part, 16, &total);   // (its barriers come after the additions)
    if (own < nk) keep[own] = mykey > prefix || (eq && s_base + rank < rem) ? 1 : 0;
}

__global__ void __launch_bounds__(256) pc_fill_u8_kernel(uint8_t *__restrict__ p, int64_t n, uint8_t v)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// Rows of at most PC_ROW_MAX kernels: a wavefront per row where the launch has at least this many rows per CU, so that the
// wavefronts fill the chip; fewer rows, and longer ones, get a workgroup each.
#define PC_ROWS_PER_CU 8
static pc_status pc_launch_rows(pc_ctx *ctx, SelBatchArg *b, const LibArg &la)
{
    if (b->n == 0) return PC_OK;
    const unsigned rows = (unsigned)b->row0[b->n];
    int cmax = 0;
    for (int i = 0; i < b->n; ++i) cmax = b->C[i] > cmax ? b->C[i] : cmax;
    if (cmax > PC_ROW_MAX) {
        const size_t lds = sizeof(uint32_t) * (size_t)cmax;
        if (rows <= (unsigned)ctx->num_cu) {
            static pc_per_device_once attr;
            if (pc_once_pending(attr, ctx->device)) {
                PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(&pc_select_long_rows_kernel<true>),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(uint32_t) * PC_ROW_LONG));
                pc_once_done(attr, ctx->device);
            }
            hipLaunchKernelGGL(pc_select_long_rows_kernel<true>, dim3(rows), dim3(1024), lds, ctx->stream, *b, la);
        } else {
            hipLaunchKernelGGL(pc_select_long_rows_kernel<false>, dim3(rows), dim3(512), lds, ctx->stream, *b, la);
        }
    } else if (rows >= (unsigned)(PC_ROWS_PER_CU * ctx->num_cu)) {
        hipLaunchKernelGGL(pc_select_rows_kernel<true>, dim3(rows), dim3(64), 0, ctx->stream, *b, la);
    } else {
        hipLaunchKernelGGL(pc_select_rows_kernel<false>, dim3(rows), dim3((unsigned)((cmax + 63) / 64 * 64)), 0, ctx->stream, *b, la);
    }
    b->n = 0;
    return pc_hip_check(ctx, hipGetLastError(), "select launch");
}

// Rows longer than PC_ROW_LONG (or few of more than PC_ROW_SPLIT), and layers ranked as a whole: scores to memory, then the
// ranking of every segment.
static pc_status pc_launch_select_segments(pc_ctx *ctx, const float *W, const float *G, int F, int C, const LibArg &la,
                                           pc_keep_mode km, int64_t n_keep, pc_score_mode sm, uint8_t *pid, uint8_t *keep)
{
    const int64_t nk = (int64_t)F * C;
    const int64_t L = (km == PC_KEEP_PER_FILTER) ? C : nk;
    const unsigned nseg = (km == PC_KEEP_PER_FILTER) ? (unsigned)F : 1u;
    if (L >= ((int64_t)1 << 31)) return pc_fail(ctx, PC_ERR_UNSUPPORTED, "select: %lld scores in one segment (limit 2^31 - 1)", (long long)L);
    // one workgroup per segment while it holds the keys in few registers, and for every row (65535 kernels at most)
    const bool rank = n_keep > 0 && n_keep < L, across = rank && km != PC_KEEP_PER_FILTER && L > PC_TOPN_WG;
    int64_t chunk = (L + PC_TOPN_CHUNKS - 1) / PC_TOPN_CHUNKS;
    chunk = chunk < 1024 ? 1024 : (chunk + 255) / 256 * 256;
    const unsigned nchunks = (unsigned)((L + chunk - 1) / chunk);
    const size_t r_bytes = (sizeof(float) * (size_t)nk + 255) / 256 * 256;
    const unsigned bin_rows = (unsigned)((nk + PC_BIN_ROW - 1) / PC_BIN_ROW);
    const size_t bin_bytes = r_bytes + (size_t)bin_rows * (PC_BIN_ROW * sizeof(uint32_t) + PC_BIN_PITCH * sizeof(uint16_t));
    // (a capture whose scratch holds the counting passes below only takes these)
    if (across && L <= PC_TOPN_BINNED && pc_scratch_ready(ctx, bin_bytes)) {
        void *scr = nullptr;
        const pc_status s = pc_scratch(ctx, bin_bytes, &scr);
        if (s != PC_OK) return s;
        uint32_t *R = (uint32_t *)scr, *K = reinterpret_cast<uint32_t *>(static_cast<unsigned char *>(scr) + r_bytes);
        uint16_t *start = reinterpret_cast<uint16_t *>(K + (size_t)bin_rows * PC_BIN_ROW);
        hipLaunchKernelGGL(pc_select_bins_kernel, dim3(bin_rows), dim3(PC_BIN_ROW), 0, ctx->stream, W, G, (int)nk, la, (int)sm, pid, R, K, start);
        hipLaunchKernelGGL(pc_topn_bins_kernel, dim3(bin_rows), dim3(PC_BIN_ROW), 0, ctx->stream, R, K, start, (int)nk, (int)n_keep, keep);
        return pc_hip_check(ctx, hipGetLastError(), "select launch");
    }
    const int nzero = across ? 3 * PC_TOPN_BINS : 0;
    void *scr = nullptr;
    pc_status s = pc_scratch(ctx, r_bytes + (across ? sizeof(uint32_t) * ((size_t)nzero + 1024 * (size_t)nchunks) : 0), &scr);
    if (s != PC_OK) return s;
    float *R = (float *)scr;
    uint32_t *hist = reinterpret_cast<uint32_t *>(static_cast<unsigned char *>(scr) + r_bytes), *chunk_hist = hist + nzero;
    const unsigned blocks = (unsigned)((nk + 255) / 256);
    hipLaunchKernelGGL(pc_select_score_kernel, dim3(blocks), dim3(256), 0, ctx->stream, W, G, nk, la, (int)sm, pid, R, hist, nzero);
    if (!rank) {
        hipLaunchKernelGGL(pc_fill_u8_kernel, dim3(blocks), dim3(256), 0, ctx->stream, keep, nk, (uint8_t)(n_keep > 0 ? 1 : 0));
    } else if (!across) {
        const int n = (int)n_keep, Li = (int)L;
        if (L <= 4096)
            hipLaunchKernelGGL(pc_topn_wg_kernel<4>, dim3(nseg), dim3(1024), 0, ctx->stream, R, Li, n, keep);
        else if (L <= 16384)
            hipLaunchKernelGGL(pc_topn_wg_kernel<16>, dim3(nseg), dim3(1024), 0, ctx->stream, R, Li, n, keep);
        else
            hipLaunchKernelGGL(pc_topn_wg_kernel<64>, dim3(nseg), dim3(1024), 0, ctx->stream, R, Li, n, keep);
    } else {
        hipLaunchKernelGGL(pc_topn_hist_kernel<0>, dim3(nchunks), dim3(256), 0, ctx->stream, R, L, chunk, (int)n_keep, hist, chunk_hist);
        hipLaunchKernelGGL(pc_topn_hist_kernel<1>, dim3(nchunks), dim3(256), 0, ctx->stream, R, L, chunk, (int)n_keep, hist, chunk_hist);
        hipLaunchKernelGGL(pc_topn_hist_kernel<2>, dim3(nchunks), dim3(256), 0, ctx->stream, R, L, chunk, (int)n_keep, hist, chunk_hist);
        hipLaunchKernelGGL(pc_topn_write_kernel, dim3(nchunks), dim3(256), 0, ctx->stream, R, L, chunk, (int)n_keep, hist, chunk_hist, keep);
    }
    return pc_hip_check(ctx, hipGetLastError(), "select launch");
}

// One layer of at most one row per CU and more than PC_ROW_SPLIT kernels per row goes through memory after all: two launches, but
// the scoring spreads over the chip (64 x 4096 10.5 us against 16.9 us, 16 x 2048 8.6 against 11.0, 256 x 4096 20.5 against 22.9;
// up to 1024 kernels, 384 rows, or 4 such layers in a call, the one launch is as fast or faster: 64 x 1024 8.8 against 8.4, 4 of
// 64 x 4096 47.8 against 23.0). Not where the scratch for it would have to be allocated during a stream capture, or cannot be: the
// other way needs none.
#define PC_ROW_SPLIT 1024
static bool pc_rows_through_memory(pc_ctx *ctx, const SelBatchArg &b)
{
    if (b.n != 1 || b.row0[1] > ctx->num_cu || b.C[0] <= PC_ROW_SPLIT) return false;
    const size_t bytes = sizeof(float) * (size_t)b.row0[1] * (size_t)b.C[0] + 256;
    return pc_scratch_ready(ctx, bytes);
}

// Layers ranked by rows go into launches of up to PC_BATCH_MAX layers, rows of at most PC_ROW_MAX kernels and longer ones apart;
// the others one by one.
pc_status pc_launch_select_batch(pc_ctx *ctx, int n, const float *const *W, const float *const *G, const int32_t *F,
                                 const int32_t *C, const LibArg &la, pc_keep_mode km, const int64_t *n_keep, pc_score_mode sm,
                                 uint8_t *const *pid, uint8_t *const *keep)
{
    SelBatchArg rows[2];
    memset(rows, 0, sizeof(rows));
    rows[0].score_mode = rows[1].score_mode = (int)sm;
    for (int l = 0; l < n; ++l) {
        pc_status s = PC_OK;
        if (km != PC_KEEP_PER_FILTER || C[l] > PC_ROW_LONG) {
            s = pc_launch_select_segments(ctx, W[l], G ? G[l] : nullptr, F[l], C[l], la, km, n_keep[l], sm, pid[l], keep[l]);
            if (s != PC_OK) return s;
            continue;
        }
        SelBatchArg &b = rows[C[l] > PC_ROW_MAX];
        const int i = b.n;
        b.W[i] = W[l]; b.G[i] = G ? G[l] : nullptr; b.C[i] = C[l];
        b.n_keep[i] = (int32_t)(n_keep[l] < C[l] ? n_keep[l] : C[l]);
        b.pid[i] = pid[l]; b.keep[i] = keep[l];
        b.row0[i + 1] = b.row0[i] + F[l];
        if (++b.n == PC_BATCH_MAX) {
            s = pc_launch_rows(ctx, &b, la);
            if (s != PC_OK) return s;
        }
    }
    pc_status s = pc_launch_rows(ctx, &rows[0], la);
    if (s != PC_OK) return s;
    const SelBatchArg &b = rows[1];
    if (pc_rows_through_memory(ctx, b))
        return pc_launch_select_segments(ctx, b.W[0], b.G[0], b.row0[1], b.C[0], la, km, b.n_keep[0], sm, b.pid[0], b.keep[0]);
    return pc_launch_rows(ctx, &rows[1], la);
}

pc_status pc_launch_select(pc_ctx *ctx, const float *W, const float *G, int F, int C, const LibArg &la,
                           pc_keep_mode km, int64_t n_keep, pc_score_mode sm, uint8_t *pid, uint8_t *keep)
{
    return pc_launch_select_batch(ctx, 1, &W, &G, &F, &C, la, km, &n_keep, sm, &pid, &keep);
}

// ------------------------------------------------------------------ packing
// Table rows are filters (row stride C, element stride 1 in the [F][C] maps) for the
// filter-major table, channels (row stride 1, element stride C) for the channel-major one.
//
// A pack of a small layer is one launch (pc_pack_one_kernel). Others are two. The first counts the kept kernels of every table row per pattern id and, for the
// matrix-core variant, writes the operand tiles (they depend on W and the masks only). The second places the
// kernels: every workgroup adds up the totals of the rows before its own, so no separate scan is needed.

// Kept kernels per pattern id, and their total, of PC_PACK_ROWS rows by one workgroup: a wavefront per row.
#define PC_PACK_ROWS 4
__device__ __forceinline__ void pc_pack_count_rows(const uint8_t *__restrict__ pid, const uint8_t *__restrict__ keep, int row0, int rows,
                                                   int len, int64_t row_stride, int64_t elem_stride, int P,
                                                   int32_t *__restrict__ grp, int32_t *__restrict__ rowtot)
{
    __shared__ int hist_all[PC_PACK_ROWS][128];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = row0 + wave;
    int *hist = hist_all[wave];
    hist[lane] = 0;
    hist[lane + 64] = 0;
    __syncthreads();
    if (row < rows) {
        int tot = 0;
#pragma unroll 4
        for (int e = lane; e < len; e += 64) {
            const int64_t k = row * row_stride + e * elem_stride;
            const int kp = keep[k], pd = pid[k];                  // both loads at once, not one behind the other
            if (kp && pd < P) { atomicAdd(&hist[pd], 1); ++tot; } // integer counts: order does not matter
        }
        for (int off = 32; off > 0; off >>= 1) tot += __shfl_down(tot, off);
        if (lane == 0) rowtot[row] = tot;
    }
    __syncthreads();
    if (row < rows)
        for (int p = lane; p < P; p += 64) grp[(int64_t)row * (PC_MAX_P + 1) + p] = hist[p];
}

// Operand tiles of one 32-filter x 32-channel block, all 9 taps.
// wz_fwd[mt][tap][ks][lane][8]: mt = filter/32, ks = channel/16; element i of lane l is
// w[f = 32*mt + l%32][c = 16*ks + 8*(l/32) + i][tap] as bf16, zero when pruned or padded.
// wz_bwd has the roles of filter and channel exchanged (rows = channels, k = filters).
// The pattern mask of a kernel comes from pid/keep, or (FROM_KINFO) from the kinfo table of an earlier pack.
#define PC_TILE_PITCH 40   // bf16 elements per LDS row: 32 + 8 keeps 16-byte alignment and spreads the banks

// 16 consecutive reduction entries of one row (bf16 bit patterns) as operands of the structured-sparse matrix
// instruction: for each of the 4 groups of 4 entries, part 1 stores the first two nonzeros and part 2 the third and
// fourth (stored value 2g + m of a part belongs to group g; an unused place holds zero), idx their 2-bit positions in
// the group: bits [4g+1:4g] and [4g+3:4g+2] for part 1, the same 16 bits higher for part 2. A place without a
// nonzero points at a position none of the part's nonzeros uses.
// ovf_pos / ovf_val (may be null): the up to 8 overflow weights (third and fourth nonzeros of a group) with their
// positions 0..15, *n_ovf their count.
__device__ __forceinline__ void pc_sparse_compress16(const uint16_t *src, uint4 *part1, uint4 *part2, uint32_t *idx,
                                                     uint32_t *ovf_pos, uint32_t *ovf_val, int *n_ovf)
{
    int no = 0;
    uint32_t w1[4] = {0u, 0u, 0u, 0u}, w2[4] = {0u, 0u, 0u, 0u};
    uint32_t ix = 0u;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        // values and positions of the nonzeros of the group, in ascending position
        uint32_t val[4] = {0u, 0u, 0u, 0u}, pos[4] = {0u, 0u, 0u, 0u};
        int n = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t u = src[4 * g + e];
            if (u & 0x7FFFu) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k == n) { val[k] = u; pos[k] = (uint32_t)e; }
                ++n;
            }
        }
#pragma unroll
        for (int k = 2; k < 4; ++k)
            if (k < n) {
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (q == no) { ovf_pos[q] = 4u * g + pos[k]; ovf_val[q] = val[k]; }
                ++no;
            }
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            const int m = n - 2 * part;                 // nonzeros left for this part
            uint32_t a = 0u, b = 0u, pa = 0u, pb = 1u;  // none: zeros at positions 0 and 1
            if (m >= 2) { a = val[2 * part]; b = val[2 * part + 1]; pa = pos[2 * part]; pb = pos[2 * part + 1]; }
            else if (m == 1) {
                const uint32_t p = pos[2 * part], x = val[2 * part];
                if (p < 3u) { a = x; pa = p; pb = 3u; } else { b = x; pa = 0u; pb = 3u; }
            }
            (part ? w2 : w1)[g] = a | (b << 16);
            ix |= (pa | (pb << 2)) << (4 * g + 16 * part);
        }
    }
    *part1 = make_uint4(w1[0], w1[1], w1[2], w1[3]);
    *part2 = make_uint4(w2[0], w2[1], w2[2], w2[3]);
    *idx = ix;
    *n_ovf = no;
}
// LDS of a tile block, shared by the bf16 and the float32 forms.
#define PC_TILE_LDS (2 * 9 * 32 * PC_TILE_PITCH * 2)
__device__ __forceinline__ unsigned char *pc_tile_lds()
{
    __shared__ __align__(16) unsigned char buf[PC_TILE_LDS];
    return buf;
}

// The 4 kernels of a 32 x 32 block that a thread brings to LDS: channel cl, filters r0 .. r0 + 3 of the block. Every thread
// loads the 9 weights of its own kernels (the 9 loads of 64 neighbours touch the same 18 cache lines), so the pattern mask
// is looked up once per kernel and no element index is divided: with contiguous loads and a mask test per element the two
// launches that build tiles took 36 us (pack) and 51 us (value update) for the 1.6 M kernels of the largest networks.
// Kernels outside the layer get mask 0. All loads are unconditional and issued before the first use.
struct PackTileRegs { unsigned m[4]; float w[4][9]; };
template <bool FROM_KINFO>
__device__ __forceinline__ void pc_pack_tile_load(const float *__restrict__ W, const uint8_t *__restrict__ pid,
                                                  const uint8_t *__restrict__ keep, const LibArg &la, const PackView &v, int fb, int cb,
                                                  PackTileRegs &t)
{
    __shared__ uint16_t lm[PC_MAX_P + 2];         // the pool's masks
    const int tid = threadIdx.x, cl = tid & 31, r0 = 4 * (tid >> 5), c = cb * 32 + cl;
    if (!FROM_KINFO && tid < la.P) lm[tid] = la.mask[tid];
    int kp[4], pd[4];
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int f = fb * 32 + r0 + i;
        const bool in = f < v.F && c < v.C;
        const int64_t k = in ? (int64_t)f * v.C + c : 0;
        if (FROM_KINFO) u[i] = v.kinfo[k];
        else { kp[i] = keep[k]; pd[i] = pid[k]; }
#pragma unroll
        for (int j = 0; j < 9; ++j) t.w[i][j] = W[k * 9 + j];
    }
    if (!FROM_KINFO) __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool in = fb * 32 + r0 + i < v.F && c < v.C;
        if (FROM_KINFO) t.m[i] = in && u[i] != 0xFFFFFFFFu ? u[i] & 511u : 0u;
        else t.m[i] = in && kp[i] && pd[i] < la.P ? lm[pd[i]] : 0u;
    }
}

// The float32 form: [row tile][tap][entry / 8][lane][4], lane l of a fragment holds row l % 32 and entries
// 4 * (l / 32) .. + 3. The block's weights are masked into LDS as they lie in W and read in both orientations.
template <bool FROM_KINFO>
__device__ __forceinline__ void pc_pack_tile_block_f32(const float *__restrict__ W, const uint8_t *__restrict__ pid,
                                                       const uint8_t *__restrict__ keep, const LibArg &la, const PackView &v,
                                                       int fb, int cb)
{
    constexpr int PITCH = 289;                    // odd: rows and columns spread over the banks
    float *tw = reinterpret_cast<float *>(pc_tile_lds());
    const int tid = threadIdx.x, cl = tid & 31, r0 = 4 * (tid >> 5);
    PackTileRegs t;
    pc_pack_tile_load<FROM_KINFO>(W, pid, keep, la, v, fb, cb, t);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 9; ++j) tw[(r0 + i) * PITCH + cl * 9 + j] = ((t.m[i] >> j) & 1u) ? t.w[i][j] : 0.0f;
    __syncthreads();
    const int KSf = v.Ck / 8, KSb = v.Fk / 8;
    float4 *of = reinterpret_cast<float4 *>(v.wz_fwd), *ob = reinterpret_cast<float4 *>(v.wz_bwd);
    for (int o = tid; o < 9 * 4 * 64; o += 256) {
        const int lane = o & 63, q = o >> 6, tap = q >> 2, ks = q & 3;
        const int row = lane & 31, e = ks * 8 + 4 * (lane >> 5);
        const float *p = tw + row * PITCH + e * 9 + tap;
        of[((int64_t)(fb * 9 + tap) * KSf + cb * 4 + ks) * 64 + lane] = make_float4(p[0], p[9], p[18], p[27]);
        const float *s = tw + e * PITCH + row * 9 + tap;
        ob[((int64_t)(cb * 9 + tap) * KSb + fb * 4 + ks) * 64 + lane] = make_float4(s[0], s[PITCH], s[2 * PITCH], s[3 * PITCH]);
    }
}

// The same, and in three parts: [row tile][tap][entry / 16][part][lane][8], lane l holds row l % 32 and entries 8 * (l / 32) .. + 7. The
// workgroups of a block have NT taps each, and with SIDES one orientation; those that share its weights follow each other on one XCD (the
// eight take workgroups in turn). Small layers are bound by the chain of a wavefront: load, LDS, split, store; large ones by their bytes, 180 a
// kernel with the float32 values (4.7 TB/s at 320 x 320). us of new values, without the parts / a workgroup per orientation / per tap / per
// three taps: 16 x 16 3.1, 4.0, 2.4, 3.0; 128 x 128 3.5, 4.4, 2.8, 3.4; 192 x 192 3.6, 4.8, 3.6, 3.9; 256 x 256 3.9, 5.4, 4.8, 4.7; 320 x 320 4.2, 6.3,
// 6.2, 5.9 (taps of a block on eight XCDs 8.1). In a pack of one launch workgroups that place rows run beside them, per orientation / tap / three
// taps: 16 x 16 4.1, 3.4, 3.5; 192 x 192 5.3, 5.8, 5.4; 256 x 256 6.8, 7.5, 7.0; 320 x 320 8.7, 8.8, 9.2.
template <bool FROM_KINFO, int NT, bool SIDES>
__device__ __forceinline__ void pc_pack_tile_parts(const float *__restrict__ W, const uint8_t *__restrict__ pid,
                                                   const uint8_t *__restrict__ keep, const LibArg &la, const PackView &v, int b)
{
    constexpr int PITCH = 33, NG = 9 / NT * (SIDES ? 2 : 1), UNITS = NT * (SIDES ? 2 : 4);    // a unit: tap, half a fragment row's entries, orientation
    static_assert(NT * 32 * PITCH * 4 <= PC_TILE_LDS, "tile");
    float *tw = reinterpret_cast<float *>(pc_tile_lds());       // [tap][filter][channel]
    const int cols = v.Cp >> 5, blocks = (v.Fp >> 5) * cols, g8 = b / (8 * NG), r8 = b - g8 * (8 * NG), n8 = blocks - 8 * g8 < 8 ? blocks - 8 * g8 : 8;
    const int part = r8 / n8, t0 = (SIDES ? part >> 1 : part) * NT, blk = 8 * g8 + r8 - part * n8, fb = blk / cols, cb = blk - fb * cols;
    const int tid = threadIdx.x, cl = tid & 31, r0 = 4 * (tid >> 5), c = cb * 32 + cl;
    __shared__ uint16_t lm[PC_MAX_P + 2];         // the pool's masks
    if (!FROM_KINFO && tid < la.P) lm[tid] = la.mask[tid];
    uint32_t u[4];
    float w[4][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int f = fb * 32 + r0 + i;
        const int64_t k = f < v.F && c < v.C ? (int64_t)f * v.C + c : 0;
        if (FROM_KINFO) u[i] = v.kinfo[k];
        else {
            const uint32_t kp = keep[k], pd = pid[k];
            u[i] = kp ? pd : 255u;                // (no id of a pool)
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) w[i][j] = W[k * 9 + t0 + j];
    }
    if (!FROM_KINFO) __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t m = 0u;
        if (fb * 32 + r0 + i < v.F && c < v.C) {
            if (FROM_KINFO) m = u[i] != 0xFFFFFFFFu ? u[i] : 0u;
            else if ((int)u[i] < la.P) m = lm[u[i]];
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) tw[(j * 32 + r0 + i) * PITCH + cl] = ((m >> (t0 + j)) & 1u) ? w[i][j] : 0.0f;
    }
    __syncthreads();
    const int lane = tid & 63, row = lane & 31, KF[2] = {v.Ck / 16, v.Fk / 16};
    uint16_t *const wz[2] = {v.wz_fwd, v.wz_bwd}, *const w3[2] = {v.w3_fwd, v.w3_bwd};
#pragma unroll
    for (int i = 0; i < (UNITS + 3) / 4; ++i) {
        const int q = i * 4 + (tid >> 6);
        if (UNITS % 4 && q >= UNITS) break;
        const int half = q & 1, j = SIDES ? q >> 1 : q >> 2;
        const bool bwd = SIDES ? part & 1 : (q >> 1) & 1;
        const int e = half * 16 + 8 * (lane >> 5), step = bwd ? PITCH : 1;
        const float *p = tw + j * 32 * PITCH + (bwd ? e * PITCH + row : row * PITCH + e);
        const int64_t fr = (int64_t)((bwd ? cb : fb) * 9 + t0 + j) * (bwd ? KF[1] : KF[0]) + (bwd ? fb : cb) * 2 + half;
        const float4 x = make_float4(p[0], p[step], p[2 * step], p[3 * step]), y = make_float4(p[4 * step], p[5 * step], p[6 * step], p[7 * step]);
        float4 *to = reinterpret_cast<float4 *>(bwd ? wz[1] : wz[0]) + fr * 128 + (lane >> 5) * 64 + row;
        to[0] = x;
        to[32] = y;
        const F32Parts s = f32_split8(x, y);
        bf16x8 *to3 = reinterpret_cast<bf16x8 *>(bwd ? w3[1] : w3[0]) + fr * 192 + lane;
#pragma unroll
        for (int k = 0; k < 3; ++k) to3[k * 64] = s.p[k];
    }
}

// How many workgroups share a block of a pack with the parts (the figures above): two, the orientations, where workgroups that place rows run
// beside them, else nine or three.
__host__ __device__ __forceinline__ int pc_tile_shares(const PackView &v, bool rows) { return rows ? 2 : v.F * v.C <= 36864 ? 9 : 3; }

// Workgroup b of a pack's operand tiles
template <bool FROM_KINFO, bool ROWS>
__device__ __forceinline__ void pc_pack_tile_block(const float *__restrict__ W, const uint8_t *__restrict__ pid,
                                                   const uint8_t *__restrict__ keep, const LibArg &la, const PackView &v, int b)
{
    if (v.w3_fwd) {
        if (ROWS) pc_pack_tile_parts<FROM_KINFO, 9, true>(W, pid, keep, la, v, b);
        else if (pc_tile_shares(v, false) == 9) pc_pack_tile_parts<FROM_KINFO, 1, false>(W, pid, keep, la, v, b);
        else pc_pack_tile_parts<FROM_KINFO, 3, false>(W, pid, keep, la, v, b);
        return;
    }
    const int fb = b / (v.Cp >> 5), cb = b - fb * (v.Cp >> 5);
    if (v.f32) return pc_pack_tile_block_f32<FROM_KINFO>(W, pid, keep, la, v, fb, cb);
    uint16_t (*tA)[32][PC_TILE_PITCH] = reinterpret_cast<uint16_t (*)[32][PC_TILE_PITCH]>(pc_tile_lds());   // [tap][filter][channel]
    uint16_t (*tB)[32][PC_TILE_PITCH] = tA + 9;                   // [tap][channel][filter]
    const int tid = threadIdx.x, cl = tid & 31, r0 = 4 * (tid >> 5);
    PackTileRegs t;
    pc_pack_tile_load<FROM_KINFO>(W, pid, keep, la, v, fb, cb, t);
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        uint32_t pr[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {             // filters r0 + 2h (low half) and r0 + 2h + 1
            const uint32_t lo = (uint32_t)-(int)((t.m[2 * h] >> j) & 1u), hi = (uint32_t)-(int)((t.m[2 * h + 1] >> j) & 1u);
            pr[h] = pc_pack_bf16x2(t.w[2 * h][j], t.w[2 * h + 1][j]) & ((lo & 0xFFFFu) | (hi & 0xFFFF0000u));
            tA[j][r0 + 2 * h][cl] = (uint16_t)pr[h];
            tA[j][r0 + 2 * h + 1][cl] = (uint16_t)(pr[h] >> 16);
        }
        *reinterpret_cast<uint2 *>(&tB[j][cl][r0]) = make_uint2(pr[0], pr[1]);
    }
    __shared__ uint32_t lflag[2];
    __shared__ uint32_t ocnt[2];                     // overflow weights of this block, forward / backward-data orientation
    __shared__ uint2 oent[2][PC_OV_SUB];
    if (tid < 2) { lflag[tid] = 0u; ocnt[tid] = 0u; }
    __syncthreads();
    const int KSf = v.Ck / 16, KSb = v.Fk / 16;
    uint4 *of = reinterpret_cast<uint4 *>(v.wz_fwd), *ob = reinterpret_cast<uint4 *>(v.wz_bwd);
    for (int o = tid; o < 9 * 2 * 64; o += 256) {
        const int lane = o & 63, q = o >> 6, tap = q >> 1, sl = q & 1;
        const int row = lane & 31, col = 16 * sl + 8 * (lane >> 5);
        if (2 * cb + sl < KSf)
            of[((int64_t)(fb * 9 + tap) * KSf + 2 * cb + sl) * 64 + lane] = *reinterpret_cast<const uint4 *>(&tA[tap][row][col]);
        if (2 * fb + sl < KSb)
            ob[((int64_t)(cb * 9 + tap) * KSb + 2 * fb + sl) * 64 + lane] = *reinterpret_cast<const uint4 *>(&tB[tap][row][col]);
    }
    // The operands of the structured-sparse instruction: this block is one step of 32 reduction entries of row tile fb
    // (forward) and of row tile cb (backward-data). Lane l of a fragment holds row l % 32 and the entries
    // 16 * (l / 32) .. + 15 of the step.
    if (!v.ws_fwd_val) return;            // uniform: only packs made for the structured-sparse kernel hold these
    const int KS32f = v.Ck / 32, KS32b = v.Fk / 32;
    for (int o = tid; o < 2 * 9 * 64; o += 256) {
        const int lane = o & 63, q = o >> 6, tap = q % 9, bwd = q / 9;
        const int rt = bwd ? cb : fb, ss = bwd ? fb : cb;
        if (ss >= (bwd ? KS32b : KS32f)) continue;
        const uint16_t *src = bwd ? &tB[tap][lane & 31][16 * (lane >> 5)] : &tA[tap][lane & 31][16 * (lane >> 5)];
        uint4 p1, p2;
        uint32_t idx, opos[8], oval[8];
        int no;
        pc_sparse_compress16(src, &p1, &p2, &idx, opos, oval, &no);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (q < no) {
                const uint32_t at = atomicAdd(&ocnt[bwd], 1u);
                if (at < PC_OV_SUB)
                    oent[bwd][at] = make_uint2(((uint32_t)tap << 11) | ((uint32_t)(lane & 31) << 6) | (16u * (lane >> 5) + opos[q]), oval[q]);
            }
        const int64_t fr = (int64_t)(rt * 9 + tap) * (bwd ? KS32b : KS32f) + ss;
        uint4 *ov = reinterpret_cast<uint4 *>(bwd ? v.ws_bwd_val : v.ws_fwd_val);
        ov[(fr * 2 + 0) * 64 + lane] = p1;
        ov[(fr * 2 + 1) * 64 + lane] = p2;
        (bwd ? v.ws_bwd_idx : v.ws_fwd_idx)[fr * 64 + lane] = idx;
        if (p2.x | p2.y | p2.z | p2.w) atomicOr(&lflag[bwd], 1u << tap);
    }
    __syncthreads();
    if (tid == 0 && cb < KS32f) v.ws_fwd_flag[(int64_t)fb * KS32f + cb] = (uint16_t)lflag[0];
    if (tid == 1 && fb < KS32b) v.ws_bwd_flag[(int64_t)cb * KS32b + fb] = (uint16_t)lflag[1];
    // The block's overflow weights, in the order of their keys (tap, row, entry): the order the atomic counter gave
    // them is not reproducible, their rank among the keys is. A list that does not fit only leaves its count.
    if (tid < 2 * PC_OV_SUB) {
        const int bwd = tid / PC_OV_SUB, e = tid % PC_OV_SUB;
        const int rt = bwd ? cb : fb, ss = bwd ? fb : cb;
        const int n = (int)ocnt[bwd];
        if (ss < (bwd ? KS32b : KS32f)) {
            const int64_t sub = (int64_t)rt * (bwd ? KS32b : KS32f) + ss;
            if (e == 0) (bwd ? v.ov_bwd_sub_cnt : v.ov_fwd_sub_cnt)[sub] = (uint32_t)n;
            if (e < n && n <= PC_OV_SUB) {
                const uint2 mine = oent[bwd][e];
                int rank = 0;
                for (int q = 0; q < n; ++q) rank += oent[bwd][q].x < mine.x;
                (bwd ? v.ov_bwd_sub_ent : v.ov_fwd_sub_ent)[sub * PC_OV_SUB + rank] = mine;
            }
        }
    }
}

// Merges the overflow lists of the two 32 x 32 blocks of a (row tile, 64-entry chunk) pair into the steps the
// structured-sparse kernel multiplies: list = blockIdx (forward lists first), 64 threads.
__device__ __forceinline__ void pc_pack_ovf_merge_body(const PackView &v, int list)
{
    __shared__ uint2 ent[2 * PC_OV_SUB];
    const int nf = (v.Fp / 32) * (v.Ck / 64);
    const bool bwd = list >= nf;
    const int l = bwd ? list - nf : list;
    const uint32_t *scnt = bwd ? v.ov_bwd_sub_cnt : v.ov_fwd_sub_cnt;
    const uint2 *sent = bwd ? v.ov_bwd_sub_ent : v.ov_fwd_sub_ent;
    uint32_t *cnt = bwd ? v.ov_bwd_cnt : v.ov_fwd_cnt;
    uint4 *oa = reinterpret_cast<uint4 *>(bwd ? v.ov_bwd_a : v.ov_fwd_a);
    uint32_t *ocol = bwd ? v.ov_bwd_col : v.ov_fwd_col;
    // sub-lists 2l and 2l + 1: the chunk's two steps of 32 entries ([rt][ss] with ss = 2 * chunk + half)
    const uint32_t n0 = scnt[2 * (int64_t)l], n1 = scnt[2 * (int64_t)l + 1];
    const int tid = threadIdx.x;
    if (n0 > PC_OV_SUB || n1 > PC_OV_SUB) {
        if (tid == 0) cnt[l] = PC_OV_BAD;
        return;
    }
    const int n = (int)(n0 + n1);
    if (tid < n) {
        const int half = tid >= (int)n0;
        uint2 e = sent[(2 * (int64_t)l + half) * PC_OV_SUB + (half ? tid - (int)n0 : tid)];
        e.x += half ? 32u : 0u;                      // entry inside the chunk
        ent[tid] = e;
    }
    __syncthreads();
    const int steps = (n + 15) / 16;
    if (tid == 0) cnt[l] = (uint32_t)steps;
    const int row = tid & 31, g = tid >> 5;
    // (the first step is always written: the kernel multiplies it without looking at the count)
    for (int s = 0; s < (steps > 1 ? steps : 1); ++s) {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int q = s * 16 + 8 * g + e;
            if (q < n) {
                const uint2 en = ent[q];
                if ((int)((en.x >> 6) & 31u) == row) w[e >> 1] |= (en.y & 0xFFFFu) << ((e & 1) * 16);
            }
        }
        oa[((int64_t)l * PC_OV_STEPS + s) * 64 + tid] = make_uint4(w[0], w[1], w[2], w[3]);
        if (tid < 16) {
            const int q = s * 16 + tid;
            uint32_t c = 0u;                         // unused columns: tap 0, entry 0 (a valid address; their weights are 0)
            if (q < n) {
                const uint32_t key = ent[q].x, tap = key >> 11;
                c = ((tap / 3u) << 12) | ((tap % 3u) << 8) | (key & 63u);
            }
            ocol[((int64_t)l * PC_OV_STEPS + s) * 16 + tid] = c;
        }
    }
}

__global__ void __launch_bounds__(64) pc_pack_ovf_merge_kernel(PackView v) { pc_pack_ovf_merge_body(v, (int)blockIdx.x); }


// First launch of a pack: the first workgroups count the filter rows, the next ncm the channel rows (gather variant, else
// none), the rest write the operand tiles (matrix-core variant), one 32 x 32 block each (with the parts of float32 weights: a share of it).
static int pc_tile_wgs(const PackView &v, bool rows) { return (v.Fp / 32) * (v.Cp / 32) * (v.w3_fwd ? pc_tile_shares(v, rows) : 1); }
static int pc_pack_row_wgs(int rows) { return (rows + PC_PACK_ROWS - 1) / PC_PACK_ROWS; }
template <bool ROWS>
__device__ __forceinline__ void pc_pack_stage1_body(const float *__restrict__ W, const uint8_t *__restrict__ pid,
                                                    const uint8_t *__restrict__ keep, const LibArg &la, const PackView &v, int ncm, int b)
{
    const int nfm = (v.F + PC_PACK_ROWS - 1) / PC_PACK_ROWS;
    if (b < nfm) {
        pc_pack_count_rows(pid, keep, b * PC_PACK_ROWS, v.F, v.C, (int64_t)v.C, 1, la.P, v.fm_grp, v.fm_rowtot);
        return;
    }
    b -= nfm;
    if (b < ncm) {
        pc_pack_count_rows(pid, keep, b * PC_PACK_ROWS, v.C, v.F, 1, (int64_t)v.C, la.P, v.cm_grp, v.cm_rowtot);
        return;
    }
    b -= ncm;
    pc_pack_tile_block<false, ROWS>(W, pid, keep, la, v, b);
}

__global__ void __launch_bounds__(256)
pc_pack_stage1_kernel(const float *__restrict__ W, const uint8_t *__restrict__ pid, const uint8_t *__restrict__ keep,
                      LibArg la, PackView v, int ncm)
{
    pc_pack_stage1_body<true>(W, pid, keep, la, v, ncm, (int)blockIdx.x);
}

// Several packs per launch: workgroup b serves block b - blk0[l] of pack l. The packs' views are read from their
// device copies (the pool is the launch's, so its size replaces the view's).
struct PackBatchArg {
    int32_t n;
    int32_t blk0[PC_BATCH_MAX + 1];
    const float *W[PC_BATCH_MAX];
    const uint8_t *pid[PC_BATCH_MAX], *keep[PC_BATCH_MAX];
    const PackView *view[PC_BATCH_MAX];
    int32_t ncm[PC_BATCH_MAX], bf16[PC_BATCH_MAX];
};

__global__ void __launch_bounds__(256) pc_pack_stage1_batch_kernel(PackBatchArg b, LibArg la)
{
    const int l = pc_batch_find(b.blk0, b.n, (int)blockIdx.x);
    const PackView v = *b.view[l];
    pc_pack_stage1_body<false>(b.W[l], b.pid[l], b.keep[l], la, v, b.ncm[l], (int)blockIdx.x - b.blk0[l]);
}

// The 4 kept weights of kernel k; taps holds the 4 tap indices, one per byte, ascending from the low byte.
__device__ __forceinline__ float4 pc_gather_taps(const float *__restrict__ W, int64_t k, uint32_t taps, bool bf16)
{
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float w = W[k * 9 + ((taps >> (8 * j)) & 255u)];
        v[j] = bf16 ? pc_bf16_to_f32(pc_f32_to_bf16(w)) : w;
    }
    return make_float4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ uint32_t pc_taps_word(const LibArg &la, int p)
{
    return (uint32_t)la.taps[p][0] | ((uint32_t)la.taps[p][1] << 8) | ((uint32_t)la.taps[p][2] << 16) | ((uint32_t)la.taps[p][3] << 24);
}

// Values again from new weights with unchanged tables, one launch for the matrix-core variant: every workgroup rebuilds the
// operand tiles of a block (masks from the kinfo table).
__global__ void __launch_bounds__(256)
pc_pack_revalue_kernel(const float *__restrict__ W, PackView v)
{
    pc_pack_tile_block<true, false>(W, nullptr, nullptr, LibArg(), v, (int)blockIdx.x);
}

// The same for several packs.
__global__ void __launch_bounds__(256) pc_pack_revalue_batch_kernel(PackBatchArg b)
{
    const int l = pc_batch_find(b.blk0, b.n, (int)blockIdx.x);
    const PackView v = *b.view[l];
    pc_pack_tile_block<true, false>(b.W[l], nullptr, nullptr, LibArg(), v, (int)blockIdx.x - b.blk0[l]);
}

// Places the kept kernels of one row at (kept kernels of the rows before) + (pattern group start) + (rank inside the group);
// the rank of an element is the number of earlier members of its group in the row, so the order inside a group is ascending.
// A workgroup per row: every wavefront ranks 64 * NE consecutive elements by ballots over the bits of their ids and leaves its
// count per pattern in LDS; one barrier later every slot is known. Everything a row needs from memory before that barrier is
// requested at once. All counts are integers, so no result depends on an execution order.
// PLACE_SLOTS: the kinfo table, all that the matrix-core kernels read (their weights are in the operand tiles; gathering the
// compact values too took 18.5 us for 3840 rows). PLACE_FM, PLACE_CM: the filter-major and channel-major tables of the
// gather kernels.
enum { PLACE_SLOTS = 0, PLACE_FM = 1, PLACE_CM = 2 };
template <int KIND>
__device__ __forceinline__ void pc_pack_place_row(const float *__restrict__ W, const uint8_t *__restrict__ pid,
                                                  const uint8_t *__restrict__ keep, int rows, int len, int64_t row_stride,
                                                  int64_t elem_stride, const LibArg &la, int bf16, const PackView &v, int row)
{
    constexpr bool FM = KIND != PLACE_CM;
    constexpr int NE = 2;                        // 512 elements of the row at a time
    __shared__ int start[128], wcnt[4][128], red[4];   // first slot of every group (less the rows before), members by wavefront
    __shared__ uint32_t ltaps[128];              // tap lists and masks of the pool
    __shared__ uint16_t lmask[128];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int P = la.P;
    int32_t *grp = (FM ? v.fm_grp : v.cm_grp) + (int64_t)row * (PC_MAX_P + 1);
    int32_t *rowptr = FM ? v.fm_rowptr : v.cm_rowptr;
    const int32_t *rowtot = FM ? v.fm_rowtot : v.cm_rowtot;
    const int idbits = P > 1 ? 32 - __builtin_clz(P - 1) : 0;
    int code[NE], rank[NE];
    auto load_codes = [&](int e0) {
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int e = e0 + (wave * NE + j) * 64 + lane, ec = e < len ? e : len - 1;
            const int64_t k = row * row_stride + ec * elem_stride;
            const int kp = keep[k], pd = pid[k];
            code[j] = e < len && kp && pd < P ? pd : 255;
        }
    };
    load_codes(0);
    if (tid < la.P) { ltaps[tid] = pc_taps_word(la, tid); lmask[tid] = la.mask[tid]; }
    int part = 0;                                // kept kernels in the rows before this one
    for (int i = tid; i < row; i += 256) part += rowtot[i];
    if (wave == 0) {
        const int n0 = lane < P ? grp[lane] : 0, n1 = lane + 64 < P ? grp[lane + 64] : 0;
        int s0 = n0, s1 = n1;                    // inclusive sums over the patterns
        for (int off = 1; off < 64; off <<= 1) {
            const int t0 = __shfl_up(s0, off), t1 = __shfl_up(s1, off);
            if (lane >= off) { s0 += t0; s1 += t1; }
        }
        start[lane] = s0 - n0;
        start[lane + 64] = __shfl(s0, 63) + s1 - n1;
    }
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off);
    if (lane == 0) red[wave] = part;
    for (int e0 = 0;;) {
        wcnt[wave][lane] = 0;
        wcnt[wave][lane + 64] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            unsigned long long same = __ballot(code[j] != 255);   // lanes of the same pattern, bit by bit of its id
            for (int bit = 0; bit < idbits; ++bit) {
                const bool on = (code[j] >> bit) & 1;
                const unsigned long long b = __ballot(on);
                same &= on ? b : ~b;
            }
            const int members = (int)__popcll(same);
            rank[j] = (int)__popcll(same & ((1ull << lane) - 1ull));
            const int before = code[j] != 255 ? wcnt[wave][code[j]] : 0;
            const bool first = rank[j] == 0;
            rank[j] += before;
            __builtin_amdgcn_wave_barrier();
            if (code[j] != 255 && first) wcnt[wave][code[j]] = before + members;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        const int base = (red[0] + red[1]) + (red[2] + red[3]);
        if (e0 == 0) {
            const int end = base + rowtot[row];
            if (KIND != PLACE_SLOTS) {
                if (tid < P) grp[tid] = base + start[tid];
                if (tid == 0) grp[P] = end;      // [P] = row end
            }
            if (tid == 0) {
                rowptr[row] = base;
                if (row == rows - 1) rowptr[rows] = end;
            }
        }
        int slot[NE];
        float4 val[NE];
        int32_t fs[NE];
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int e = e0 + (wave * NE + j) * 64 + lane, ec = e < len ? e : len - 1;
            const int64_t k = row * row_stride + ec * elem_stride;
            const int c = code[j] != 255 ? code[j] : 0;
            slot[j] = base + start[c] + rank[j];
            for (int w = 0; w < wave; ++w) slot[j] += wcnt[w][c];
            if (KIND != PLACE_SLOTS && code[j] != 255) val[j] = pc_gather_taps(W, k, ltaps[c], bf16 != 0);
            fs[j] = FM ? 0 : v.slot_of[k];
        }
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int e = e0 + (wave * NE + j) * 64 + lane;
            const int64_t k = row * row_stride + e * elem_stride;
            if (e >= len) continue;
            const bool kept = code[j] != 255;
            if (KIND == PLACE_SLOTS) {
                v.kinfo[k] = kept ? ((uint32_t)slot[j] << 9) | lmask[code[j]] : 0xFFFFFFFFu;
            } else if (FM) {
                v.slot_of[k] = kept ? slot[j] : -1;
                if (kept) {
                    v.fm_c[slot[j]] = (uint16_t)e;
                    v.fm_pid[slot[j]] = (uint8_t)code[j];
                    v.slot_f[slot[j]] = (uint16_t)row;
                    v.fm_val[slot[j]] = val[j];
                }
            } else if (kept) {
                v.cm_f[slot[j]] = (uint16_t)e;
                v.cm_slot[slot[j]] = fs[j];
                v.cm_val[slot[j]] = val[j];
            }
        }
        e0 += 256 * NE;
        if (e0 >= len) break;
        load_codes(e0);
        __syncthreads();
        if (tid < P) start[tid] += (wcnt[0][tid] + wcnt[1][tid]) + (wcnt[2][tid] + wcnt[3][tid]);
        __syncthreads();
    }
}

template <int KIND>
__global__ void __launch_bounds__(256)
pc_pack_place_kernel(const float *__restrict__ W, const uint8_t *__restrict__ pid, const uint8_t *__restrict__ keep,
                     int rows, int len, int64_t row_stride, int64_t elem_stride, LibArg la, int bf16, PackView v)
{
    pc_pack_place_row<KIND>(W, pid, keep, rows, len, row_stride, elem_stride, la, bf16, v, (int)blockIdx.x);
}

template <int KIND> __global__ void __launch_bounds__(256) pc_pack_place_batch_kernel(PackBatchArg b, LibArg la)
{
    const int l = pc_batch_find(b.blk0, b.n, (int)blockIdx.x);
    const PackView v = *b.view[l];
    const int row = (int)blockIdx.x - b.blk0[l];
    if constexpr (KIND == PLACE_CM)
        pc_pack_place_row<KIND>(b.W[l], b.pid[l], b.keep[l], v.C, v.F, (int64_t)1, (int64_t)v.C, la, b.bf16[l], v, row);
    else
        pc_pack_place_row<KIND>(b.W[l], b.pid[l], b.keep[l], v.F, v.C, (int64_t)v.C, (int64_t)1, la, b.bf16[l], v, row);
}

// A pack of the matrix-core kernels in one launch: the first F workgroups place a row each, the rest write the operand tiles. A row of
// up to 512 kernels is ranked at once, so its pattern groups are known without a counting launch, and the kept kernels before it are
// counted from the masks themselves, 16 at a time, by every workgroup again (128 KiB of each mask at most, from L2).
// Bound by latency: 256 x 256 8.5 us in two launches, 5.9 in one; 256 x 512 9.3, 7.8; 400 x 400 10.1, 9.8; 512 x 512 10.7, 13.5.
#define PC_PACK_ONE 131072
__device__ __forceinline__ int pc_count_kept(uint32_t keep, uint32_t pid, uint32_t ge)
{
    const uint32_t kept = ((keep & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | keep, past = ((pid & 0x7F7F7F7Fu) + ge) | pid;   // bit 7 of every byte
    return __popc(kept & ~past & 0x80808080u);
}

__device__ __forceinline__ void pc_pack_place_counted(const uint8_t *__restrict__ pid, const uint8_t *__restrict__ keep, const LibArg &la,
                                                      const PackView &v, int row)
{
    __shared__ int start[128], wcnt[4][128], red[4];
    __shared__ uint16_t lmask[128];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int P = la.P, C = v.C, idbits = P > 1 ? 32 - __builtin_clz(P - 1) : 0;
    int code[2], rank[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int e = (wave * 2 + j) * 64 + lane, k = row * C + (e < C ? e : C - 1);
        const int kp = keep[k], pd = pid[k];
        code[j] = e < C && kp && pd < P ? pd : 255;
    }
    if (tid < P) lmask[tid] = la.mask[tid];
    const int before = row * C, whole = before >> 4;
    const uint32_t ge = (uint32_t)(128 - P) * 0x01010101u;
    int part = 0;
#pragma unroll 4
    for (int i = tid; i < whole; i += 256) {
        const uint4 k = reinterpret_cast<const uint4 *>(keep)[i], p = reinterpret_cast<const uint4 *>(pid)[i];
        part += pc_count_kept(k.x, p.x, ge) + pc_count_kept(k.y, p.y, ge) + pc_count_kept(k.z, p.z, ge) + pc_count_kept(k.w, p.w, ge);
    }
    if (16 * whole + tid < before) part += keep[16 * whole + tid] && pid[16 * whole + tid] < P;
    wcnt[wave][lane] = 0;
    wcnt[wave][lane + 64] = 0;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        unsigned long long same = __ballot(code[j] != 255);   // lanes of the same pattern, bit by bit of its id
        for (int bit = 0; bit < idbits; ++bit) {
            const bool on = (code[j] >> bit) & 1;
            const unsigned long long b = __ballot(on);
            same &= on ? b : ~b;
        }
        rank[j] = (int)__popcll(same & ((1ull << lane) - 1ull));
        const int ahead = code[j] != 255 ? wcnt[wave][code[j]] : 0;
        const bool first = rank[j] == 0;
        rank[j] += ahead;
        __builtin_amdgcn_wave_barrier();
        if (code[j] != 255 && first) wcnt[wave][code[j]] = ahead + (int)__popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off);
    if (lane == 0) red[wave] = part;
    __syncthreads();
    const int base = (red[0] + red[1]) + (red[2] + red[3]);
    if (wave == 0) {
        const int n0 = (wcnt[0][lane] + wcnt[1][lane]) + (wcnt[2][lane] + wcnt[3][lane]);
        const int n1 = (wcnt[0][lane + 64] + wcnt[1][lane + 64]) + (wcnt[2][lane + 64] + wcnt[3][lane + 64]);
        int s0 = n0, s1 = n1;                    // inclusive sums over the patterns
        for (int off = 1; off < 64; off <<= 1) {
            const int t0 = __shfl_up(s0, off), t1 = __shfl_up(s1, off);
            if (lane >= off) { s0 += t0; s1 += t1; }
        }
        const int half = __shfl(s0, 63), end = base + half + __shfl(s1, 63);
        start[lane] = s0 - n0;
        start[lane + 64] = half + s1 - n1;
        if (lane == 0) {
            v.fm_rowptr[row] = base;
            if (row == v.F - 1) v.fm_rowptr[v.F] = end;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int e = (wave * 2 + j) * 64 + lane;
        if (e >= C) continue;
        const bool kept = code[j] != 255;
        const int c = kept ? code[j] : 0;
        int slot = base + start[c] + rank[j];
        for (int w = 0; w < wave; ++w) slot += wcnt[w][c];
        v.kinfo[row * C + e] = kept ? ((uint32_t)slot << 9) | lmask[c] : 0xFFFFFFFFu;
    }
}

__global__ void __launch_bounds__(256)
pc_pack_one_kernel(const float *__restrict__ W, const uint8_t *__restrict__ pid, const uint8_t *__restrict__ keep, LibArg la, PackView v)
{
    const int b = (int)blockIdx.x;
    if (b < v.F) pc_pack_place_counted(pid, keep, la, v, b);
    else pc_pack_tile_block<false, true>(W, pid, keep, la, v, b - v.F);
}

// Re-gathers values with unchanged tables (one thread per kernel (f,c)).
__global__ void __launch_bounds__(256)
pc_pack_regather_fm_kernel(const float *__restrict__ W, LibArg la, int bf16, PackView v)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)v.F * v.C) return;
    int slot = v.slot_of[k];
    if (slot < 0) return;
    v.fm_val[slot] = pc_gather_taps(W, k, pc_taps_word(la, v.fm_pid[slot]), bf16 != 0);
}

__global__ void __launch_bounds__(256) pc_pack_regather_cm_kernel(PackView v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= v.cm_rowptr[v.C]) return;
    v.cm_val[i] = v.fm_val[v.cm_slot[i]];
}

// The overflow lists of a pack made for the structured-sparse kernel (no-op for other packs).
static int pc_ovf_lists(const PackView &v) { return v.ov_fwd_cnt ? (v.Fp / 32) * (v.Ck / 64) + (v.Cp / 32) * (v.Fk / 64) : 0; }
static void pc_launch_ovf_merge(pc_ctx *ctx, const PackView &v)
{
    const int n = pc_ovf_lists(v);
    if (n > 0) hipLaunchKernelGGL(pc_pack_ovf_merge_kernel, dim3((unsigned)n), dim3(64), 0, ctx->stream, v);
}

// The same for several packs in one launch.
__global__ void __launch_bounds__(64) pc_pack_ovf_merge_batch_kernel(PackBatchArg b)
{
    const int l = pc_batch_find(b.blk0, b.n, (int)blockIdx.x);
    pc_pack_ovf_merge_body(*b.view[l], (int)blockIdx.x - b.blk0[l]);
}

static void pc_launch_ovf_merge_batch(pc_ctx *ctx, int m, pc_packed *const *pk)
{
    PackBatchArg a;
    memset(&a, 0, sizeof(a));
    a.n = m;
    for (int i = 0; i < m; ++i) {
        a.view[i] = pk[i]->v_dev;
        a.blk0[i + 1] = a.blk0[i] + pc_ovf_lists(pk[i]->v);
    }
    if (a.blk0[m] > 0) hipLaunchKernelGGL(pc_pack_ovf_merge_batch_kernel, dim3((unsigned)a.blk0[m]), dim3(64), 0, ctx->stream, a);
}

pc_status pc_launch_pack(pc_ctx *ctx, pc_packed *pk, const float *W, const uint8_t *pid, const uint8_t *keep)
{
    PackView v = pk->v;
    LibArg la;
    pc_fill_lib(&la, pk->lib, v.P);
    int bf16 = pk->dtype == PC_BF16;
    hipStream_t st = ctx->stream;
    const bool mfma = pk->variant == PC_VARIANT_MFMA;
    // the channel-major table serves the gather kernels' backward-data pass (the matrix-core kernels read operand tiles)
    const int nfm = pc_pack_row_wgs(v.F), ncm = mfma ? 0 : pc_pack_row_wgs(v.C);
    const int ntiles = mfma ? pc_tile_wgs(v, true) : 0;
    if (mfma && v.C <= 512 && (int64_t)v.F * v.C <= PC_PACK_ONE && (((uintptr_t)pid | (uintptr_t)keep) & 15) == 0) {
        hipLaunchKernelGGL(pc_pack_one_kernel, dim3((unsigned)(v.F + ntiles)), dim3(256), 0, st, W, pid, keep, la, v);
        pc_launch_ovf_merge(ctx, v);
        return pc_hip_check(ctx, hipGetLastError(), "pack launch");
    }
    hipLaunchKernelGGL(pc_pack_stage1_kernel, dim3((unsigned)(nfm + ncm + ntiles)), dim3(256), 0, st, W, pid, keep, la, v, ncm);
    if (mfma) {
        hipLaunchKernelGGL(pc_pack_place_kernel<PLACE_SLOTS>, dim3((unsigned)v.F), dim3(256), 0, st, W, pid, keep, v.F, v.C,
                           (int64_t)v.C, (int64_t)1, la, bf16, v);
    } else {
        hipLaunchKernelGGL(pc_pack_place_kernel<PLACE_FM>, dim3((unsigned)v.F), dim3(256), 0, st, W, pid, keep, v.F, v.C,
                           (int64_t)v.C, (int64_t)1, la, bf16, v);
        hipLaunchKernelGGL(pc_pack_place_kernel<PLACE_CM>, dim3((unsigned)v.C), dim3(256), 0, st, W, pid, keep, v.C, v.F, (int64_t)1,
                           (int64_t)v.C, la, bf16, v);
    }
    pc_launch_ovf_merge(ctx, v);
    return pc_hip_check(ctx, hipGetLastError(), "pack launch");
}

// Re-packs several handles with one pool: two launches per group of up to PC_BATCH_MAX packs (four when some use the
// gather kernels).
pc_status pc_launch_pack_batch(pc_ctx *ctx, int n, pc_packed *const *pk, const float *const *W, const uint8_t *const *pid,
                               const uint8_t *const *keep, const LibArg &la)
{
    for (int l0 = 0; l0 < n; l0 += PC_BATCH_MAX) {
        const int m = n - l0 < PC_BATCH_MAX ? n - l0 : PC_BATCH_MAX;
        PackBatchArg s1, sl, fm, cm;
        memset(&s1, 0, sizeof(s1));
        s1.n = m;
        for (int i = 0; i < m; ++i) {
            const pc_packed *p = pk[l0 + i];
            const bool mfma = p->variant == PC_VARIANT_MFMA;
            s1.W[i] = W[l0 + i]; s1.pid[i] = pid[l0 + i]; s1.keep[i] = keep[l0 + i];
            s1.view[i] = p->v_dev;
            s1.ncm[i] = mfma ? 0 : pc_pack_row_wgs(p->v.C);
            s1.bf16[i] = p->dtype == PC_BF16;
        }
        sl = s1;
        fm = s1;
        cm = s1;
        for (int i = 0; i < m; ++i) {
            const pc_packed *p = pk[l0 + i];
            const bool mfma = p->variant == PC_VARIANT_MFMA;
            s1.blk0[i + 1] = s1.blk0[i] + pc_pack_row_wgs(p->v.F) + s1.ncm[i] + (mfma ? pc_tile_wgs(p->v, false) : 0);
            sl.blk0[i + 1] = sl.blk0[i] + (mfma ? p->v.F : 0);
            fm.blk0[i + 1] = fm.blk0[i] + (mfma ? 0 : p->v.F);
            cm.blk0[i + 1] = cm.blk0[i] + (mfma ? 0 : p->v.C);
        }
        hipLaunchKernelGGL(pc_pack_stage1_batch_kernel, dim3((unsigned)s1.blk0[m]), dim3(256), 0, ctx->stream, s1, la);
        if (sl.blk0[m] > 0)
            hipLaunchKernelGGL(pc_pack_place_batch_kernel<PLACE_SLOTS>, dim3((unsigned)sl.blk0[m]), dim3(256), 0, ctx->stream, sl, la);
        if (fm.blk0[m] > 0) {
            hipLaunchKernelGGL(pc_pack_place_batch_kernel<PLACE_FM>, dim3((unsigned)fm.blk0[m]), dim3(256), 0, ctx->stream, fm, la);
            hipLaunchKernelGGL(pc_pack_place_batch_kernel<PLACE_CM>, dim3((unsigned)cm.blk0[m]), dim3(256), 0, ctx->stream, cm, la);
        }
        pc_launch_ovf_merge_batch(ctx, m, pk + l0);
        pc_status s = pc_hip_check(ctx, hipGetLastError(), "pack (several layers) launch");
        if (s != PC_OK) return s;
    }
    return PC_OK;
}

// Matrix-core packs share launches of up to PC_BATCH_MAX; gather-kernel packs are updated one by one.
pc_status pc_launch_update_values_batch(pc_ctx *ctx, int n, pc_packed *const *pk, const float *const *W)
{
    PackBatchArg b;
    memset(&b, 0, sizeof(b));
    pc_packed *bpk[PC_BATCH_MAX];
    auto flush = [&]() -> pc_status {
        if (b.n == 0) return PC_OK;
        hipLaunchKernelGGL(pc_pack_revalue_batch_kernel, dim3((unsigned)b.blk0[b.n]), dim3(256), 0, ctx->stream, b);
        pc_launch_ovf_merge_batch(ctx, b.n, bpk);
        b.n = 0;
        return pc_hip_check(ctx, hipGetLastError(), "update_values (several layers) launch");
    };
    for (int l = 0; l < n; ++l) {
        pc_packed *p = pk[l];
        if (p->variant != PC_VARIANT_MFMA) {
            pc_status s = pc_launch_update_values(ctx, p, W[l]);
            if (s != PC_OK) return s;
            continue;
        }
        const int i = b.n;
        bpk[i] = p;
        b.W[i] = W[l];
        b.view[i] = p->v_dev;
        b.blk0[i + 1] = b.blk0[i] + pc_tile_wgs(p->v, false);
        if (++b.n == PC_BATCH_MAX) {
            pc_status s = flush();
            if (s != PC_OK) return s;
        }
    }
    return flush();
}

pc_status pc_launch_update_values(pc_ctx *ctx, pc_packed *pk, const float *W)
{
    PackView v = pk->v;
    if (pk->variant == PC_VARIANT_MFMA) {
        hipLaunchKernelGGL(pc_pack_revalue_kernel, dim3((unsigned)pc_tile_wgs(v, false)), dim3(256), 0, ctx->stream, W, v);
        pc_launch_ovf_merge(ctx, v);
    } else {
        LibArg la;
        pc_fill_lib(&la, pk->lib, v.P);
        const int bf16 = pk->dtype == PC_BF16;
        const unsigned blocks = (unsigned)(((int64_t)v.F * v.C + 255) / 256);
        hipLaunchKernelGGL(pc_pack_regather_fm_kernel, dim3(blocks), dim3(256), 0, ctx->stream, W, la, bf16, v);
        hipLaunchKernelGGL(pc_pack_regather_cm_kernel, dim3(blocks), dim3(256), 0, ctx->stream, v);
    }
    return pc_hip_check(ctx, hipGetLastError(), "update_values launch");
}

// dense[f][c][t] = value of the kept tap, 0 elsewhere. The 9 values of a workgroup's 256 kernels go through LDS, so that the
// stores are contiguous. The slots come from the kinfo table of a matrix-core pack or the tables of a gather-kernel pack;
// compact == nullptr (the latter only): the pack's own values.
template <bool KINFO>
__global__ void __launch_bounds__(256)
pc_scatter_kernel(const float *__restrict__ compact, float *__restrict__ dense, LibArg la, PackView v)
{
    __shared__ __align__(16) float s[256 * 9];
    const int tid = threadIdx.x;
    const int64_t nk = (int64_t)v.F * v.C, k0 = (int64_t)blockIdx.x * 256, k = k0 + tid < nk ? k0 + tid : nk - 1;
    int slot = -1;
    unsigned m = 0u;
    if (KINFO) {
        const uint32_t u = v.kinfo[k];
        if (u != 0xFFFFFFFFu) { slot = (int)(u >> 9); m = u & 511u; }
    } else {
        slot = v.slot_of[k];
        if (slot >= 0) m = la.mask[v.fm_pid[slot]];
    }
    float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
    if (slot >= 0) val = compact ? reinterpret_cast<const float4 *>(compact)[slot] : v.fm_val[slot];
    int j = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const bool on = (m >> t) & 1u;
        s[tid * 9 + t] = !on ? 0.0f : j == 0 ? val.x : j == 1 ? val.y : j == 2 ? val.z : val.w;
        j += on;
    }
    __syncthreads();
    const int n = nk - k0 < 256 ? (int)(nk - k0) * 9 : 256 * 9;
    float *dst = dense + k0 * 9;
    if ((reinterpret_cast<uintptr_t>(dense) & 15) == 0) {
#pragma unroll
        for (int i = tid; i < 256 * 9 / 4; i += 256)
            if (i * 4 + 3 < n) reinterpret_cast<float4 *>(dst)[i] = reinterpret_cast<const float4 *>(s)[i];
        const int i = (n & ~3) + tid;
        if (i < n) dst[i] = s[i];
    } else {
        for (int i = tid; i < n; i += 256) dst[i] = s[i];
    }
}

// The own values of a matrix-core pack: they are in the operand tiles of the forward pass, zeros included. One 32-filter x
// 32-channel block per workgroup, fragments in, rows of 32 * 9 floats out.
__global__ void __launch_bounds__(256) pc_unpack_tiles_kernel(float *__restrict__ dense, PackView v, int tiles_c)
{
    constexpr int PITCH = 289;                    // odd: rows and columns spread over the banks
    __shared__ float s[32 * PITCH];
    const int tid = threadIdx.x, fb = (int)blockIdx.x / tiles_c, cb = (int)blockIdx.x - fb * tiles_c;
    if (v.f32) {
        const float4 *in = reinterpret_cast<const float4 *>(v.wz_fwd);
        float4 q[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {             // tap i, 8-entry step tid / 64
            const int ks = cb * 4 + (tid >> 6);
            q[i] = ks < v.Ck / 8 ? in[((int64_t)(fb * 9 + i) * (v.Ck / 8) + ks) * 64 + (tid & 63)] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            float *d = s + (tid & 31) * PITCH + ((tid >> 6) * 8 + 4 * ((tid >> 5) & 1)) * 9 + i;
            d[0] = q[i].x; d[9] = q[i].y; d[18] = q[i].z; d[27] = q[i].w;
        }
    } else {
        const uint4 *in = reinterpret_cast<const uint4 *>(v.wz_fwd);
        uint4 q[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {             // fragment (tap, 16-entry step) i * 4 + tid / 64 of 18
            const int fr = i * 4 + (tid >> 6), tap = fr >> 1, ks = cb * 2 + (fr & 1);
            q[i] = fr < 18 && ks < v.Ck / 16 ? in[((int64_t)(fb * 9 + tap) * (v.Ck / 16) + ks) * 64 + (tid & 63)] : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int fr = i * 4 + (tid >> 6);
            if (fr >= 18) break;
            float *d = s + (tid & 31) * PITCH + ((fr & 1) * 16 + 8 * ((tid >> 5) & 1)) * 9 + (fr >> 1);
            const uint32_t w[4] = {q[i].x, q[i].y, q[i].z, q[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                d[18 * e] = __uint_as_float(w[e] << 16);
                d[18 * e + 9] = __uint_as_float(w[e] & 0xFFFF0000u);
            }
        }
    }
    __syncthreads();
    const int nrows = v.F - fb * 32 < 32 ? v.F - fb * 32 : 32, ncols = v.C - cb * 32 < 32 ? v.C - cb * 32 : 32;
    for (int r = tid >> 6; r < nrows; r += 4)
        for (int j = tid & 63; j < ncols * 9; j += 64) dense[((int64_t)(fb * 32 + r) * v.C + cb * 32) * 9 + j] = s[r * PITCH + j];
}

pc_status pc_launch_scatter(pc_ctx *ctx, const pc_packed *pk, const float *compact, float *dense, int from_pack)
{
    const PackView v = pk->v;
    const bool mfma = pk->variant == PC_VARIANT_MFMA;
    if (mfma && from_pack) {
        const int tiles_c = (v.C + 31) / 32;
        hipLaunchKernelGGL(pc_unpack_tiles_kernel, dim3((unsigned)((v.F + 31) / 32 * tiles_c)), dim3(256), 0, ctx->stream, dense, v, tiles_c);
        return pc_hip_check(ctx, hipGetLastError(), "unpack launch");
    }
    LibArg la;
    pc_fill_lib(&la, pk->lib, v.P);
    const unsigned blocks = (unsigned)(((int64_t)v.F * v.C + 255) / 256);
    if (mfma) hipLaunchKernelGGL(pc_scatter_kernel<true>, dim3(blocks), dim3(256), 0, ctx->stream, compact, dense, la, v);
    else hipLaunchKernelGGL(pc_scatter_kernel<false>, dim3(blocks), dim3(256), 0, ctx->stream, from_pack ? nullptr : compact, dense, la, v);
    return pc_hip_check(ctx, hipGetLastError(), "scatter launch");
}
