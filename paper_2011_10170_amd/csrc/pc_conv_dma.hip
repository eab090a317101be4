// Forward / backward-data at stride 1 on the matrix cores, both operands brought to LDS by direct loads (see pc_conv_mfma.hip
// for the implicit-GEMM formulation, the operand tiles and the MFMA register layout).
#include "pc_mfma.h"
#include <math.h>

// A workgroup of 4 wavefronts owns 64 output channels x (32 rows x 1, 2 or 4 columns per wavefront); two workgroups share a CU.
// The reduction runs in chunks of 32 input channels: the weights of a chunk (36 KiB) and the input tile with its border are
// loaded straight into the workgroup's one LDS buffer, and all of the chunk's matrix instructions follow from there. One
// workgroup loads (or stores a finished tile) while the other multiplies; a wavefront's priority rises through a chunk, so
// that of two workgroups that multiply at the same time the one ahead finishes first and the two fall out of step by
// themselves.
//   Rows: the rows of all images, N * H of them, in order. The staged tile is rows of "padded images" of H + 1 rows (one zero
//     row between two images), so a tile covers any 32, 64 or 128 rows without a gap, whatever the map's height.
//   Columns: the 32 lanes of a B fragment are 32 rows of one column, so the fragment of column j is the operand of tap column s
//     for output column j - s: a tap row of a wavefront's 4 columns reads 6 fragments for its 24 matrix instructions beside the 6 of
//     the weights.
//   LDS: a staged row is its columns' 64 bytes and one 16-byte element more, so lanes a row apart start in different banks.
// In the kernel that keeps the weights in registers (pc_conv_mfma_ws.hip) each of the four multiplying wavefronts requests the same
// fragments, 64 B/clk of vector-cache hits, and nothing is multiplied while a tile is stored.

#define DM_KC 32                     // input channels per chunk
#define DM_NA 36                     // direct loads (1 KiB) of the weights per chunk: 2 row tiles x 9 taps x 2 k-steps
#define DM_NB 11                     // of the input tile per wavefront at most
#define DM_A_BYTES (DM_NA * 1024)
#define DM_OOB 0x80000000u           // past the end of any tensor taken here, also with a chunk's offset added
#define DM_LDS_MAX (80 * 1024)       // two workgroups per CU
#define DM_STG 144                   // bytes per pixel (64 channels) where a finished tile passes through LDS

// The tile's columns and staged columns for 1, 2 or 4 columns per wavefront.
struct DmaGeo {
    int32_t IW, EPR, nB;             // staged columns, 16-byte elements per staged row, direct loads of the input tile
    uint32_t mg_EPR;
};

struct DmaArgs {
    int32_t N, H, W, in_CH, out_CH;  // the output map has the input map's extent
    int32_t KS, nch;                 // k-steps of 16 per tap in the operand tiles; chunks
    int32_t flip;                    // position t of the 3 x 3 neighbourhood takes weight tap 8 - t (backward-data)
    int32_t lgCG;                    // log2 of the wavefronts side by side in a tile's columns; the others lie below each other
    int32_t TR, nrow, rows;          // rows of a tile, staged rows, N * H
    int32_t m_fast, fdiv, tiles_x;   // tile index = slow * fdiv + fast, as in MfmaArgs; column tiles of the widest part
    // Parts of the list of tiles: end[2], end[1], end[0] are the tiles of 4, 2 and 1 columns per wavefront up to which a part
    // runs; tile t of a part lies where tile t >> 1 of the part with twice the columns would.
    int32_t lgB, end[3];
    uint32_t in_bytes, out_bytes, wz_bytes;
    uint32_t mg_fd, mg_tx, mg_H, mg_H1;
    DmaGeo geo[3];                   // by log2 of the columns per wavefront
    const uint16_t *act_mask;
};

// 64 lanes x 16 bytes from a buffer to the 1 KiB of LDS at lds_off; an offset past the buffer's end writes zeros. As inline
// assembly because the compiler orders every later LDS read behind a direct load it knows of: here the wait is one
// s_waitcnt in front of a barrier.
__device__ __forceinline__ void dm_load(const v4u32 &rsrc, int voff, int soff, int lds_off)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// The words of a buffer resource (what __builtin_amdgcn_make_buffer_rsrc builds, as an operand of inline assembly).
__device__ __forceinline__ v4u32 dm_rsrc(const void *p, uint32_t bytes)
{
    const uint64_t a = (uint64_t)p;
    const v4u32 r = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu)),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
    return r;
}

struct DmaTile { int mt, r0, x0; };  // tile of 64 output channels, first row, first column

struct DmaWave {
    int lane, w, cg, rg, G;
    v4u32 xs, ws;
    int a_voff;
    uint32_t voff[DM_NB];            // byte offsets of this lane's elements of the input tile, first chunk
    uint32_t part;                   // two bits per element: which 8 of the chunk's 32 channels
};

// Tile t of the part with 1 << lg columns per wavefront.
__device__ __forceinline__ DmaTile dm_tile(const DmaArgs &g, int t, int lg)
{
    const int sh = g.lgB - lg;
    const uint32_t p = (uint32_t)t >> sh;
    const uint32_t tq = pc_udiv(p, g.mg_fd), trm = p - tq * g.fdiv;
    const uint32_t pt = g.m_fast ? tq : trm;
    const uint32_t rt = pc_udiv(pt, g.mg_tx);
    DmaTile o;
    o.mt = (int)(g.m_fast ? trm : tq);
    o.r0 = (int)rt * g.TR;
    o.x0 = (int)(((pt - rt * g.tiles_x) << sh) + ((uint32_t)t & ((1u << sh) - 1u))) << (lg + g.lgCG);
    return o;
}

// The elements of a tile that this lane loads: element e of the tile is the 16-byte part e % EPR of staged row e / EPR.
__device__ __forceinline__ void dm_offsets(DmaWave &s, const DmaArgs &g, const DmaGeo &q, const DmaTile &t)
{
    const int V0 = t.r0 + (int)pc_udiv((uint32_t)t.r0, g.mg_H);
    s.part = 0;
#pragma unroll
    for (int k = 0; k < DM_NB; ++k) {
        const uint32_t e = (uint32_t)((s.w + 4 * k) * 64 + s.lane);
        const uint32_t row = pc_udiv(e, q.mg_EPR), rem = e - row * q.EPR;
        const uint32_t v = V0 + row;
        const int n = (int)pc_udiv(v, g.mg_H1);
        const int y = (int)v - n * (g.H + 1) - 1, x = t.x0 - 1 + (int)(rem >> 2);
        const bool ok = (int)row < g.nrow && (int)(rem >> 2) < q.IW && y >= 0 && n < g.N && (unsigned)x < (unsigned)g.W;
        s.voff[k] = ok ? (uint32_t)((n * g.H + y) * g.W + x) * (uint32_t)(g.in_CH * 2) + (rem & 3u) * 16u : DM_OOB;
        s.part |= (rem & 3u) << (2 * k);
    }
}

__device__ __forceinline__ void dm_issue(const DmaWave &s, const DmaArgs &g, int nB, int mt, int ch)
{
    // Fragment f of the chunk: row tile f & 1, tap position (f / 2) % 9, k-step f / 18. A lane takes the row whose number has bits 2
    // and 3 exchanged: 8 of its 16 accumulators are then 8 consecutive output channels.
    // (the wavefront's number is hidden from the compiler here: it would compute all scalar offsets ahead and spill them)
    int w = s.w;
    asm volatile("" : "+s"(w));
#pragma unroll
    for (int k = 0; k < DM_NA / 4; ++k) {
        const int f = w + 4 * k, t = (f >> 1) % 9, kk = f / 18;
        dm_load(s.ws, s.a_voff, (((mt * 2 + (f & 1)) * 9 + (g.flip ? 8 - t : t)) * g.KS + ch * 2 + kk) * 1024, f * 1024);
    }
    const bool cut = ch == g.nch - 1 && (g.in_CH & (DM_KC - 1));      // channels past the last one are zeros
    const uint32_t parts = (uint32_t)(g.in_CH & (DM_KC - 1)) >> 3;
#pragma unroll
    for (int k = 0; k < DM_NB; ++k) {
        const int b = w + 4 * k;
        if (b < nB) {
            uint32_t vo = s.voff[k];
            if (cut) vo = ((s.part >> (2 * k)) & 3u) >= parts ? DM_OOB : vo;
            dm_load(s.xs, (int)vo, ch * (DM_KC * 2), DM_A_BYTES + b * 1024);
        }
    }
}

// The matrix instructions of one chunk; pa, pb: this lane's first weight and input fragment, RP: bytes per staged row. The
// fragments of a tap are read during the one before it, the input fragments of a tap row during the one before.
template <int BT>
__device__ __forceinline__ void dm_chunk(f32x16 (&acc)[2][BT], const unsigned char *pa, const unsigned char *pb, int RP)
{
    constexpr int HB = (BT + 3) / 2;   // the fragments of the next tap row are read in two parts
    bf16x8 aq[2][2], bq[2][BT + 2];
#pragma unroll
    for (int c = 0; c < BT + 2; ++c) bq[0][c] = *reinterpret_cast<const bf16x8 *>(pb + c * 64);
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) aq[0][ii] = *reinterpret_cast<const bf16x8 *>(pa + ii * 1024);
#pragma unroll
    for (int t = 0; t < 18; ++t) {
        const int rr = t / 3, s = t % 3;
        if (t == 6) __builtin_amdgcn_s_setprio(1);
        if (t == 12) __builtin_amdgcn_s_setprio(2);
        if (t < 17) {
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) aq[(t + 1) & 1][ii] = *reinterpret_cast<const bf16x8 *>(pa + ((t + 1) * 2 + ii) * 1024);
        }
        if (rr < 5 && s < 2) {
#pragma unroll
            for (int c = s * HB; c < (s + 1) * HB && c < BT + 2; ++c)
                bq[(rr + 1) & 1][c] = *reinterpret_cast<const bf16x8 *>(pb + ((rr + 1) % 3) * RP + c * 64 + ((rr + 1) / 3) * 32);
        }
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int j = 0; j < BT; ++j)
                acc[ii][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[t & 1][ii], bq[rr & 1][j + s], acc[ii][j], 0, 0, 0);
#pragma unroll
        for (int m = 0; m < 2 * BT; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  // one matrix instruction
            __builtin_amdgcn_sched_group_barrier(0x100, BT == 1 ? 2 : 1, 0);    // LDS reads
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The tiles first, first + G, ... < end of the part with BT = 1 << LG columns per wavefront. fresh: nothing has used LDS yet.
template <int LG, int ACT>
__device__ __forceinline__ void dm_part(DmaWave &s, const DmaArgs &g, unsigned char *lds, __amdgpu_buffer_rsrc_t osrc, __amdgpu_buffer_rsrc_t msrc,
                                        int first, int end, bool &fresh)
{
    constexpr int BT = 1 << LG;
    const DmaGeo q = g.geo[LG];
    const int RP = q.EPR * 16;
    for (int ti = first; ti < end; ti += s.G) {
        const DmaTile t = dm_tile(g, ti, LG);
        dm_offsets(s, g, q, t);
        // rows past the last one are multiplied with the last one's operands and not stored
        const int row = t.r0 + s.rg * 32 + (s.lane & 31), rowc = row < g.rows ? row : g.rows - 1;
        const int lrow = rowc + (int)pc_udiv((uint32_t)rowc, g.mg_H) - (t.r0 + (int)pc_udiv((uint32_t)t.r0, g.mg_H));
        const unsigned char *pa = lds + s.lane * 16, *pb = lds + DM_A_BYTES + lrow * RP + (s.lane >> 5) * 16 + s.cg * (BT * 64);
        f32x16 acc[2][BT];
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int j = 0; j < BT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[ii][j][r] = 0.0f;
        for (int ch = 0; ch < g.nch; ++ch) {
            if (!fresh) asm volatile("s_barrier" ::: "memory");      // every wavefront has read what the loads replace
            fresh = false;
            __builtin_amdgcn_s_setprio(3);
            dm_issue(s, g, q.nB, t.mt, ch);
            __builtin_amdgcn_s_setprio(0);
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
            dm_chunk<BT>(acc, pa, pb, RP);
        }
        // The tile leaves through LDS, 32 rows x 2 columns of a wavefront at a time, so that 8 lanes store the 128 bytes of a pixel.
        __builtin_amdgcn_s_setprio(3);
        asm volatile("s_barrier" ::: "memory");
        constexpr int NC = BT == 1 ? 1 : 2, NP = NC * 4;
        unsigned char *stg = lds + s.w * (64 * DM_STG);
#pragma unroll
        for (int h = 0; h < BT / NC; ++h) {
            v4u32 mk[NP];
            uint32_t off[NP];
#pragma unroll
            for (int it = 0; it < NP; ++it) {
                const int px = it * 8 + (s.lane >> 3);
                const int orow = t.r0 + s.rg * 32 + (px & 31), x = t.x0 + s.cg * BT + h * NC + (px >> 5), m = t.mt * 64 + (s.lane & 7) * 8;
                off[it] = orow < g.rows && x < g.W && m < g.out_CH ? (uint32_t)(orow * g.W + x) * (uint32_t)(g.out_CH * 2) + (uint32_t)(m * 2) : DM_OOB;
                if (ACT == PC_ACT_RELU_MASK) mk[it] = __builtin_amdgcn_raw_buffer_load_b128(msrc, (int)off[it], 0, 0);
            }
#pragma unroll
            for (int jj = 0; jj < NC; ++jj)
#pragma unroll
                for (int e = 0; e < 4; ++e) {       // accumulators 8 * (e & 1) .. + 7 of row tile e >> 1: channels 16 * e + 8 * (lane / 32) .. + 7
                    v4u32 pv;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        pv[u] = pc_pack_bf16x2(acc[e >> 1][h * NC + jj][(e & 1) * 8 + 2 * u], acc[e >> 1][h * NC + jj][(e & 1) * 8 + 2 * u + 1]);
                    *reinterpret_cast<v4u32 *>(stg + (jj * 32 + (s.lane & 31)) * DM_STG + e * 32 + (s.lane >> 5) * 16) = pv;
                }
#pragma unroll
            for (int it = 0; it < NP; ++it) {
                v4u32 pv = *reinterpret_cast<const v4u32 *>(stg + (it * 8 + (s.lane >> 3)) * DM_STG + (s.lane & 7) * 16);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (ACT == PC_ACT_RELU) pv[u] = pc_relu_bf16x2(pv[u]);
                    if (ACT == PC_ACT_RELU_MASK) pv[u] = pc_mask_bf16x2(pv[u], mk[it][u]);
                }
                __builtin_amdgcn_raw_buffer_store_b128(pv, osrc, (int)off[it], 0, 0);
            }
        }
    }
}

template <int LG, int ACT>
__global__ void __launch_bounds__(256, 2)
pc_mfma_conv_dma_kernel(const uint16_t *__restrict__ in, uint16_t *__restrict__ out, const uint16_t *__restrict__ wz, DmaArgs g)
{
    extern __shared__ __align__(16) unsigned char lds[];
    DmaWave s;
    s.lane = threadIdx.x & 63;
    s.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    s.cg = s.w & ((1 << g.lgCG) - 1);
    s.rg = s.w >> g.lgCG;
    s.G = gridDim.x;
    int vb = blockIdx.x;
    if ((s.G & 7) == 0) vb = (blockIdx.x & 7) * (s.G >> 3) + (blockIdx.x >> 3);   // neighbours in the tile order share an XCD
    s.xs = dm_rsrc(in, g.in_bytes);
    s.ws = dm_rsrc(wz, g.wz_bytes);
    s.a_voff = ((s.lane & ~12) | ((s.lane & 4) << 1) | ((s.lane & 8) >> 1)) * 16;
    const __amdgpu_buffer_rsrc_t osrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, g.out_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t msrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(ACT == PC_ACT_RELU_MASK ? g.act_mask : out), 0, g.out_bytes, 0x00020000);
    bool fresh = true;
    if constexpr (LG >= 2) dm_part<2, ACT>(s, g, lds, osrc, msrc, vb, g.end[2], fresh);
    dm_part<1, ACT>(s, g, lds, osrc, msrc, 2 * g.end[2] + vb, g.end[1], fresh);
    dm_part<0, ACT>(s, g, lds, osrc, msrc, 2 * g.end[1] + vb, g.end[0], fresh);
}

// ---- plan and launch

// Fills the plan for 1 << lgB columns per wavefront and 1 << lgCG wavefronts side by side; false when it does not fit.
static bool plan_dma(const MfmaArgs &g, bool flip, int lgB, int lgCG, DmaArgs *out, size_t *lds, int *grid, double *est, int num_cu)
{
    DmaArgs t;
    memset(&t, 0, sizeof(t));
    t.N = g.N; t.H = g.in_H; t.W = g.in_W; t.in_CH = g.in_CH; t.out_CH = g.out_CH;
    t.KS = g.KS; t.nch = (g.in_CH + DM_KC - 1) / DM_KC; t.flip = flip;
    t.lgCG = lgCG; t.lgB = lgB;
    t.TR = 32 * (4 >> lgCG);
    const int64_t rows = (int64_t)g.N * g.in_H;
    if ((rows + g.N + 2 * t.TR) * (g.in_H + 1) >= ((int64_t)1 << 32) || rows >= (1 << 24)) return false;   // multiply-high divisions stay exact
    t.rows = (int)rows;
    // image boundaries inside a tile (tiles start at multiples of TR)
    int cross = g.in_H % t.TR == 0 ? 0 : t.TR % g.in_H == 0 ? t.TR / g.in_H - 1 : (t.TR - 1 + g.in_H - 1) / g.in_H;
    if (cross > g.N - 1) cross = g.N - 1;
    t.nrow = t.TR + 2 + cross;
    for (int l = 0; l <= lgB; ++l) {
        DmaGeo &q = t.geo[l];
        q.IW = (1 << (l + lgCG)) + 2;
        q.EPR = (DM_KC / 8) * q.IW + 1;
        q.mg_EPR = pc_udiv_magic(q.EPR);
        q.nB = (t.nrow * q.EPR + 63) / 64;
    }
    const int nB = t.geo[lgB].nB, TC = 1 << (lgB + lgCG);
    *lds = (size_t)DM_A_BYTES + (size_t)nB * 1024;
    if (nB > 4 * DM_NB || *lds > DM_LDS_MAX) return false;
    t.tiles_x = (g.in_W + TC - 1) / TC;
    const int64_t p_tiles = (rows + t.TR - 1) / t.TR * t.tiles_x;
    const int m_tiles = (g.out_CH + 63) / 64;
    const int64_t total = p_tiles * m_tiles;
    const int64_t in_bytes = rows * g.in_W * g.in_CH * 2, out_bytes = rows * g.in_W * g.out_CH * 2;
    if (total > (1 << 28) || in_bytes >= ((int64_t)1 << 31) || out_bytes >= ((int64_t)1 << 31)) return false;
    t.in_bytes = (uint32_t)in_bytes; t.out_bytes = (uint32_t)out_bytes;
    t.wz_bytes = (uint32_t)((size_t)((g.out_CH + 127) / 128 * 4) * 9 * t.KS * 1024);
    t.m_fast = in_bytes >= (int64_t)g.out_CH * g.in_CH * 18;     // neighbours share the larger operand
    t.fdiv = t.m_fast ? m_tiles : (int)p_tiles;
    if (total * (t.fdiv > t.tiles_x ? t.fdiv : t.tiles_x) >= ((int64_t)1 << 32)) return false;
    t.mg_fd = pc_udiv_magic(t.fdiv); t.mg_tx = pc_udiv_magic(t.tiles_x);
    t.mg_H = pc_udiv_magic(g.in_H); t.mg_H1 = pc_udiv_magic(g.in_H + 1);
    t.act_mask = g.act_mask;
    // Estimated time (us). A round is one tile for each of the workgroups the chip holds, two per CU; a last round of at most one
    // tile per CU has each CU's whole rate for its tiles. A tile takes its chunks, each a fixed time and one for its direct loads of
    // the input, and an end; the tensors take their bytes (the input with its border, in pieces of 64) at 4.5 TB/s, what these
    // loads reach where the tensors come from memory and not, as in a loop over one layer, from the last cache (there 7). Constants for
    // 4, 2 and 1 columns per wavefront from 1790 timings of 127 layer shapes (1 to 125 images, 4 x 4 to 224 x 224, 8 to 512
    // channels; 7 % rms; the plan with the least estimate is on average 2 % slower than the fastest of a shape).
    // What is left over after whole rounds of the widest tiles goes to narrower ones where that is estimated to end earlier:
    // 56 x 56, 256 -> 256, batch 32 is 784 tiles of 4 columns for 512 workgroups; 512 of them, 512 of 2 columns and 64 of 1
    // column take 85.6 us instead of 90.5, 14 x 14, 512 -> 512 32.4 instead of 54.
    static const double kPair[3][3] = {{1.288, 0.0127, 1.86}, {2.116, 0.0166, 2.111}, {2.082, 0.0672, 3.27}};    // chunk, direct load, tile
    static const double kOne[3][3] = {{0.977, 0.0134, 0.953}, {1.311, 0.0149, 1.433}, {2.337, 0.0113, 2.546}};
    const int slots = num_cu * 2;
    double best = 1e30;
    int64_t most = 0;
    for (int o = 0; o < 4; ++o) {     // o & 1: the first part ends with its last whole round, o & 2: so does the second
        int64_t n[3] = {0, 0, 0}, left = total, m = 0;
        double cost = 0.0;
        for (int l = lgB; l >= 0; --l) {
            n[l] = l > 0 && (o & (l == lgB ? 1 : 2)) ? left / slots * slots : left;
            if (n[l] > m) m = n[l];
            left = (left - n[l]) * 2;
            const int64_t rem = n[l] % slots;
            const bool one = rem > 0 && rem <= num_cu;
            cost += (double)(n[l] / slots + (rem > num_cu)) * (t.nch * (kPair[l][0] + kPair[l][1] * t.geo[l].nB) + kPair[l][2]);
            if (one) cost += t.nch * (kOne[l][0] + kOne[l][1] * t.geo[l].nB) + kOne[l][2];
        }
        if (cost < best) {
            best = cost;
            most = m;
            t.end[2] = (int)n[2];
            t.end[1] = (int)(2 * n[2] + n[1]);
            t.end[0] = (int)(2 * t.end[1] + n[0]);
        }
    }
    const double move = 2.0 * ((double)p_tiles * t.nrow * (TC + 2) * (g.in_CH < DM_KC ? DM_KC : g.in_CH) + (double)rows * g.in_W * g.out_CH) / 4.5e6;
    *est = 4.08 + pow(pow(best, 2.22) + pow(move, 2.22), 1.0 / 2.22);
    *grid = (int)(most < slots ? most : slots);
    *out = t;
    return true;
}

template <int LG, int ACT>
static hipError_t launch_dma_act(int device, hipStream_t st, int grid, size_t lds, const uint16_t *in, uint16_t *out, const uint16_t *wz, const DmaArgs &g)
{
    static pc_per_device_once attr;
    if (pc_once_pending(attr, device)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&pc_mfma_conv_dma_kernel<LG, ACT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, DM_LDS_MAX);
        if (e != hipSuccess) return e;
        pc_once_done(attr, device);
    }
    hipLaunchKernelGGL((pc_mfma_conv_dma_kernel<LG, ACT>), dim3((unsigned)grid), dim3(256), lds, st, in, out, wz, g);
    return hipGetLastError();
}

template <int LG>
static hipError_t launch_dma(int device, hipStream_t st, int grid, size_t lds, const uint16_t *in, uint16_t *out, const uint16_t *wz, const DmaArgs &g, int act)
{
    if (act == PC_ACT_RELU) return launch_dma_act<LG, PC_ACT_RELU>(device, st, grid, lds, in, out, wz, g);
    if (act == PC_ACT_RELU_MASK) return launch_dma_act<LG, PC_ACT_RELU_MASK>(device, st, grid, lds, in, out, wz, g);
    return launch_dma_act<LG, PC_ACT_NONE>(device, st, grid, lds, in, out, wz, g);
}

// pcfg: -1 or 40 / 41 (2 / 4 columns per wavefront). *launched stays false where the kernel does not take the launch or its
// estimate is not below limit (us).
pc_status pc_run_mfma_conv_dma(pc_ctx *ctx, int pcfg, double limit, const MfmaArgs &g0, bool flip, const uint16_t *in, uint16_t *out, const uint16_t *wz,
                               bool *launched, int act)
{
    *launched = false;
    if (g0.lstep != 1 || g0.oscale != 1 || (g0.in_CH & 7) || (g0.out_CH & 7)) return PC_OK;
    DmaArgs best;
    size_t best_lds = 0;
    int best_grid = 0, best_b = -1;
    double best_est = limit;
    for (int b = 1; b <= 2; ++b) {
        if (pcfg >= 0 && pcfg != 39 + b) continue;
        for (int lg = 0; lg <= 2; ++lg) {
            DmaArgs t;
            size_t lds;
            int grid;
            double est;
            if (!plan_dma(g0, flip, b, lg, &t, &lds, &grid, &est, ctx->num_cu)) continue;
            if (est < best_est) { best = t; best_lds = lds; best_grid = grid; best_b = b; best_est = est; }
        }
    }
    if (best_b < 0) return PC_OK;
    const hipError_t e = best_b == 2 ? launch_dma<2>(ctx->device, ctx->stream, best_grid, best_lds, in, out, wz, best, act)
                                     : launch_dma<1>(ctx->device, ctx->stream, best_grid, best_lds, in, out, wz, best, act);
    *launched = true;
    pc_note_kernel(ctx, "pc_mfma_conv_dma_kernel<%d, %d>", best_b, act);
    return pc_hip_check(ctx, e, "MFMA conv (direct loads) launch");
}
