// Forward / backward-data on the matrix cores, both operands brought to LDS by direct loads (see pc_conv_mfma.hip
// for the implicit-GEMM formulation, the operand tiles and the MFMA register layout).
#include "pc_dma.h"
#include <algorithm>

#include <math.h>
#include <type_traits>

// A workgroup of 4 wavefronts owns 64 output channels x 64 columns of 16 rows (fewer columns in the narrower forms). The reduction runs
// in chunks of 32 input channels: the weights of a chunk (36 KiB) and the input tile with its border are loaded straight into an
// LDS buffer, and all of the chunk's matrix instructions follow from there.
//   Instruction: v_mfma_f32_16x16x32_bf16. The rate the chip holds depends on what the operands and sums toggle: fed from LDS with
//     pruned weights and ReLU outputs 2.28 PFLOP/s against 2.0 with v_mfma_f32_32x32x16_bf16 (2.38 for both on zeros).
//   Two ways of hiding the loads. Large layers (pc_mfma_conv_dma_kernel): one buffer, and two workgroups share a CU: one loads (or
//     stores a finished tile) while the other multiplies; a wavefront's priority rises through a chunk, so that of two workgroups
//     that multiply at the same time the one ahead finishes first and the two fall out of step by themselves. Layers of a few tiles
//     per CU (pc_mfma_conv_solo_kernel): a workgroup has the CU to itself, with two or three buffers and wavefronts that only load.
//   Rows: the rows of all images, N * H of them, in order, so a tile covers any 16, 32 or 64 rows without a gap, whatever the map's
//     height. Stride 1: they are staged as they follow each other, and where a row's neighbour lies outside its image the lane reads
//     zeros behind the staged rows. Stride 2: the staged tile is rows of "padded images" of H + 1 rows (one zero row between two images).
//   Columns: the 16 columns of a B operand are 16 rows of one column of the map, so the fragment of column j is the operand of tap
//     column s for output column j - s: the three taps of a row read BT + 2 fragments for BT columns.
//   LDS: a staged row is its columns' 64 bytes and two 16-byte elements more where there is room. ds_read_b128 takes 16 lanes at a time,
//     0 to 3, 12 to 15 and 20 to 27 first: those rows of one 16-byte group of channels and the other rows of the next group, which stand in
//     16 different places of 256 bytes exactly if a row is twice an odd number of elements long. (With one element more every read took twice the
//     time, with an image's end among the 16 rows and a row of zeros there three times. A zero is read from the place of the
//     256 bytes where the row would have stood.) us with one element and rows of
//     zeros -> here, tiles of 64 x 128: 64 images 7 x 7 512 -> 512 16.1 -> 14.1, 128 images 8 x 8 256 -> 256 10.2 -> 9.3; of 64 x 256: 64 images 14 x 14
//     256 -> 256 15.5 -> 14.3, 32 images 512 -> 512 27.3 -> 26.1; tiles of two workgroups per CU, where LDS was busy half of the time, 1 to 3 %.
// In the kernel that keeps the weights in registers (pc_conv_mfma_ws.hip) each of the four multiplying wavefronts requests the same
// fragments, 64 B/clk of vector-cache hits, and nothing is multiplied while a tile is stored.

#define DM_KC 32                     // input channels per chunk
#define DM_NA 36                     // direct loads (1 KiB) of the weights per chunk: 9 taps x 4 fragments of 16 output channels
#define DM_NB 11                     // of the input tile per wavefront at most
#define DM_A_BYTES (DM_NA * 1024)
#define DM_LDS_MAX (160 * 1024)
#define DM_STG 144                   // bytes per pixel (64 channels) where a finished tile passes through LDS

// Direct loads of the input tile per wavefront where every wavefront has as many (three buffers)
constexpr __host__ __device__ int dm_nbw(int bt) { return bt == 2 ? 3 : 4; }

// What a kernel computes. The tiles of the stride-2 passes lie on the output gradient's map (the forward pass's output).
//   DM_FWD2: rows 2y, 2y + 1, 2y + 2 of a padded image go into output row y. Even and odd rows are staged apart, so that 16 output rows
//     still read 16 staged rows next to each other; 2 * BT + 1 fragments serve the three taps of a row.
//   DM_BWD2: input row 2y takes tap row 1 from output row y, row 2y + 1 tap row 2 from y and tap row 0 from y + 1, columns alike. A tile's
//     four parity classes of pixels are summed together, from BT + 1 fragments per row.
enum { DM_S1 = 0, DM_FWD2 = 1, DM_BWD2 = 2 };

// The tap of step t of a chunk, in the order in which the fragments of a row are used up.
template <int MODE> constexpr __host__ __device__ int dm_tap(int t)
{
    constexpr int order[9] = {3, 4, 5, 6, 7, 8, 1, 2, 0};
    return MODE == DM_BWD2 ? order[t] : t;
}

// Staged columns for a tile width
struct DmaGeo {
    int32_t IW, EPR, nB, zero;       // staged columns, 16-byte elements per staged row, direct loads of the input tile, where zeros stand behind it (bytes)
    uint32_t mg_EPR;
};

struct DmaArgs {
    int32_t N, H, W, in_CH, out_CH;  // H x W: the map of the tiles
    int32_t in_H, in_W, out_H, out_W;
    int32_t KS, nch;                 // k-steps of 16 per tap in the operand tiles; chunks
    int32_t flip;                    // position t of the 3 x 3 neighbourhood takes weight tap 8 - t (backward-data)
    int32_t lgCG;                    // log2 of the wavefronts side by side in a tile's columns; the others lie below each other
    int32_t TR, nrow, rows;          // rows of a tile, staged rows (of a parity at stride 2 forward), N * H
    int32_t m_fast, fdiv, tiles_x;   // tile index = slow * fdiv + fast, as in MfmaArgs; column tiles
    // The list of tiles: `rounds` whole rounds (a tile for every workgroup), then `last` tiles, one each for the first workgroups, and
    // the remaining tiles cut into 1 << lgP pieces of their columns, one each for the workgroups after those
    int32_t rounds, last, pieces, lgP;
    int32_t share, apart;            // workgroups that ask an L2 for a row tile's weights ahead, each for its part (0: none do); their distance
    uint32_t in_bytes, out_bytes, wz_bytes, buf_bytes;
    uint32_t mg_fd, mg_tx, mg_H, mg_H1;
    DmaGeo geo[3];                   // whole tiles, halves, quarters
    const uint16_t *act_mask;
};

struct DmaTile { int mt, r0, x0; };  // tile of 64 output channels, first row, first column

struct DmaRows { const unsigned char *p[3]; };

struct DmaWave {
    int lane, w, cg, rg;
    v4u32 xs, ws;
    int a_voff;
    uint32_t voff[DM_NB];            // byte offsets of this lane's elements of the input tile, first chunk
    uint32_t part;                   // two bits per element: which 8 of the chunk's 32 channels
};

// Piece t of tiles of BT columns per wavefront cut into 1 << sh pieces.
template <int BT>
__device__ __forceinline__ DmaTile dm_tile(const DmaArgs &g, int t, int sh)
{
    const uint32_t p = (uint32_t)t >> sh;
    const uint32_t tq = pc_udiv(p, g.mg_fd), trm = p - tq * g.fdiv;
    const uint32_t pt = g.m_fast ? tq : trm;
    const uint32_t rt = pc_udiv(pt, g.mg_tx);
    DmaTile o;
    o.mt = (int)(g.m_fast ? trm : tq);
    o.r0 = (int)rt * g.TR;
    o.x0 = (int)(((pt - rt * g.tiles_x) * BT + ((uint32_t)t & ((1u << sh) - 1u)) * (BT >> sh)) << g.lgCG);
    return o;
}

// The elements of a tile that this lane loads (NBW > 0: NBW of them): element e of the tile is the 16-byte part e % EPR of staged row e / EPR.
// ASK: and asks for the first chunk of each at once, into the buffer at lb (with all offsets made first a launch's first pixels were asked for 0.4
// to 1 us later).
template <int MODE, int NBW, bool ASK = false>
__device__ __forceinline__ void dm_offsets(DmaWave &s, const DmaArgs &g, const DmaGeo &q, const DmaTile &t, int lb = 0)
{
    const uint32_t parts = g.nch == 1 && (g.in_CH & (DM_KC - 1)) ? (uint32_t)(g.in_CH & (DM_KC - 1)) >> 3 : 4u;
    const int V0 = MODE == DM_S1 ? t.r0 - 1 : t.r0 + (int)pc_udiv((uint32_t)t.r0, g.mg_H);
    s.part = 0;
    int lane = s.lane;      // (hidden from the compiler: it would keep the quotients of all elements from tile to tile, in scratch)
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int k = 0; k < (NBW ? NBW : DM_NB); ++k) {
        if (!NBW && s.w + 4 * k >= q.nB) break;
        const uint32_t e = (uint32_t)((s.w + 4 * k) * 64 + lane);
        const uint32_t row = pc_udiv(e, q.mg_EPR), rem = e - row * q.EPR;
        const int c = (int)(rem >> 2);
        if (MODE == DM_S1) {
            const int v = V0 + (int)row, x = t.x0 - 1 + c;
            const bool ok = (int)row < g.nrow && c < q.IW && (unsigned)v < (unsigned)g.rows && (unsigned)x < (unsigned)g.in_W;
            s.voff[k] = ok ? (uint32_t)(v * g.in_W + x) * (uint32_t)(g.in_CH * 2) + (rem & 3u) * 16u : DM_OOB;
        } else {
            const int odd = MODE == DM_FWD2 && (int)row >= g.nrow;
            const uint32_t v = V0 + row - (odd ? g.nrow : 0);
            const int n = (int)pc_udiv(v, g.mg_H1);
            int y = (int)v - n * (g.H + 1);
            if (MODE == DM_FWD2) y = 2 * y + odd - 1;
            const int x = MODE == DM_FWD2 ? 2 * t.x0 - 1 + c : t.x0 + c;
            const bool ok = (int)row < (MODE == DM_FWD2 ? 2 * g.nrow : g.nrow) && c < q.IW && (unsigned)y < (unsigned)g.in_H && n < g.N &&
                            (unsigned)x < (unsigned)g.in_W;
            s.voff[k] = ok ? (uint32_t)((n * g.in_H + y) * g.in_W + x) * (uint32_t)(g.in_CH * 2) + (rem & 3u) * 16u : DM_OOB;
        }
        s.part |= (rem & 3u) << (2 * k);
        if (ASK) dm_load(s.xs, (int)((rem & 3u) >= parts ? DM_OOB : s.voff[k]), 0, lb + (s.w + 4 * k) * 1024);
    }
}

// The direct loads of chunk ch of a tile (its offsets are in s) into the buffer at lb by wavefront s.w of four: fragment s.w of every tap
// position and every fourth load of the input tile (nB of them; NBW > 0: NBW for every wavefront).
//   AT = 4: a wavefront multiplies all 64 channels of the tile. Row m of fragment a is output channel 16 * (m / 4) + 4 * a + m % 4 of the
//     tile, so that a lane's sums are 16 consecutive channels.
//   AT = 2: half of them. Row m of fragment 2 * h + a is channel 32 * h + 8 * (m / 4) + 4 * a + m % 4: 8 consecutive channels.
template <int AT>
__device__ __forceinline__ int dm_weight_offset(const DmaArgs &g, int lane)     // of a lane in a fragment
{
    const int m = lane & 15, kg = lane >> 4, at = (kg >> 1) * 1024 + (kg & 1) * 512;
    return AT == 4 ? at + (m >> 3) * (9 * 1024) * g.KS + (16 * ((m >> 2) & 1) + (m & 3)) * 16 : at + (8 * (m >> 2) + (m & 3)) * 16;
}

template <int MODE, int AT, int FR>
__device__ __forceinline__ void dm_issue_weights(const DmaWave &s, const DmaArgs &g, int w, int mt, int ch, int lb)
{
    const int first = AT == 4 ? w * 64 : (w >> 1) * (9 * 1024) * g.KS + (w & 1) * 64;
    if constexpr (FR == 4) {
#pragma unroll
        for (int t = 0; t < 9; ++t)
            dm_load(s.ws, s.a_voff, ((mt * 18 + (MODE == DM_S1 && g.flip ? 8 - t : dm_tap<MODE>(t))) * g.KS + ch * 2) * 1024 + first, lb + (t * 4 + w) * 1024);
    } else {               // the first 32 channels: fragment w % 2 of taps w / 2, w / 2 + 2, ..
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int t = 2 * i + (w >> 1);
            if (t < 9) dm_load(s.ws, s.a_voff, ((mt * 18 + (g.flip ? 8 - t : t)) * g.KS + ch * 2) * 1024 + (w & 1) * 64, lb + (t * 2 + (w & 1)) * 1024);
        }
    }
}

template <int NBW>
__device__ __forceinline__ void dm_issue_input(const DmaWave &s, const DmaArgs &g, int w, int nB, int ch, int lb)
{
    const bool cut = ch == g.nch - 1 && (g.in_CH & (DM_KC - 1));      // channels past the last one are zeros
    const uint32_t parts = (uint32_t)(g.in_CH & (DM_KC - 1)) >> 3;
#pragma unroll
    for (int k = 0; k < (NBW ? NBW : DM_NB); ++k) {
        const int b = w + 4 * k;
        if (NBW || b < nB) {
            uint32_t vo = s.voff[k];
            if (cut) vo = ((s.part >> (2 * k)) & 3u) >= parts ? DM_OOB : vo;
            dm_load(s.xs, (int)vo, ch * (DM_KC * 2), lb + b * 1024);
        }
    }
}

// The matrix instructions of one chunk; pa: this lane's first weight fragment, pb: its first input fragments in the order in which the
// tap rows are used. The weight fragments of a tap are read one tap ahead (two or three where a tap is 8 or 4
// instructions); the input fragments of the next tap row replace those of this one as its last tap has used them.
template <int MODE, int AT, int BT, int FR = 4>
__device__ __forceinline__ void dm_chunk(f32x4 (&acc)[AT][MODE == DM_BWD2 ? 4 * BT : BT], const unsigned char *pa, const DmaRows &pb)
{
    constexpr int D = AT * BT <= 4 ? 3 : AT * BT <= 8 ? 2 : 1, NF = MODE == DM_S1 ? BT + 2 : MODE == DM_FWD2 ? 2 * BT + 1 : BT + 1;
    bf16x8 aq[D + 1][AT], bq[NF];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int a = 0; a < AT; ++a) aq[d][a] = *reinterpret_cast<const bf16x8 *>(pa + (d * FR + a) * 1024);
#pragma unroll
    for (int c = 0; c < NF; ++c) bq[c] = *reinterpret_cast<const bf16x8 *>(pb.p[0] + c * 64);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int r = dm_tap<MODE>(t) / 3, q = dm_tap<MODE>(t) % 3;
        const bool refill = t == 5 || (t == 2 && MODE != DM_BWD2);
        const unsigned char *pn = pb.p[t < 3 ? 1 : 2];                      // the next tap row
        const int cls = MODE == DM_BWD2 ? ((r != 1) * 2 + (q != 1)) * BT : 0;
        auto read = [&](int c) { bq[c] = *reinterpret_cast<const bf16x8 *>(pn + c * 64); };
        if (t == 3) __builtin_amdgcn_s_setprio(1);
        if (t == 6) __builtin_amdgcn_s_setprio(2);
        if (refill) {      // those that the row's last tap does not use
            if (MODE == DM_BWD2) read(BT);
            else { read(0); read(1); }
        }
#pragma unroll
        for (int j = 0; j < BT; ++j) {
            if (t + D < 9) {
#pragma unroll
                for (int a = j * AT / BT; a < (j + 1) * AT / BT; ++a)
                    aq[(t + D) % (D + 1)][a] = *reinterpret_cast<const bf16x8 *>(pa + ((t + D) * FR + a) * 1024);
            }
            const int c = MODE == DM_S1 ? j + q : MODE == DM_FWD2 ? 2 * j + q : j + (q == 0);
#pragma unroll
            for (int a = 0; a < AT; ++a) acc[a][cls + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq[t % (D + 1)][a], bq[c], acc[a][cls + j], 0, 0, 0);
            if (refill) {
                read(c);
                if (MODE == DM_FWD2 && j + 1 < BT) read(c + 1);
            }
        }
        // (in program order: reads go into the shadow of the matrix instructions one at a time)
        if (refill) __builtin_amdgcn_sched_group_barrier(0x100, MODE == DM_BWD2 ? 1 : 2, 0);
#pragma unroll
        for (int j = 0; j < BT; ++j) {
            if (t + D < 9 && (j + 1) * AT / BT > j * AT / BT) __builtin_amdgcn_sched_group_barrier(0x100, BT < AT ? AT / BT : 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, AT, 0);
            if (refill && MODE == DM_FWD2 && j + 1 < BT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            else if (refill) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Where a lane of a wavefront reads a tile: byte offsets in an input buffer of the three tap rows (stride 2: of the staged row).
template <int MODE, int BT>
__device__ __forceinline__ void dm_lane_rows(const DmaWave &s, const DmaArgs &g, const DmaGeo &q, const DmaTile &t, int (&at)[3])
{
    // rows past the last one are multiplied with the last one's operands and not stored
    const int row = t.r0 + s.rg * 16 + (s.lane & 15), rowc = row < g.rows ? row : g.rows - 1, RP = q.EPR * 16;
    const int n = (int)pc_udiv((uint32_t)rowc, g.mg_H), left = (s.lane >> 4) * 16 + s.cg * (BT * (MODE == DM_FWD2 ? 128 : 64));
    if (MODE == DM_S1) {
        const int y = rowc - n * g.H;
        at[0] = (rowc - t.r0) * RP + left; at[1] = at[0] + RP; at[2] = at[1] + RP;
        if (y == 0) at[0] = q.zero + (at[0] & 255);
        if (y == g.H - 1) at[2] = q.zero + (at[2] & 255);
    } else {
        at[0] = (rowc + n - (t.r0 + (int)pc_udiv((uint32_t)t.r0, g.mg_H))) * RP + left;
        at[1] = at[0] + (MODE == DM_FWD2 ? g.nrow * RP : RP);
        at[2] = at[0] + RP;
    }
}

__device__ __forceinline__ DmaRows dm_rows(const unsigned char *buf, const int (&at)[3]) { return {{buf + at[0], buf + at[1], buf + at[2]}}; }

// A wavefront's sums of a finished tile go out through the LDS at stg (of this wavefront alone): 64 pixels at a time, so that 8 lanes
// store the 128 bytes of a pixel.
// Output offset of the 16 bytes that this lane stores in step it of the columns from j0 on (DM_BWD2: of parity class CLS).
template <int MODE, int AT, int BT, int CLS>
__device__ __forceinline__ uint32_t dm_out_offset(const DmaWave &s, const DmaArgs &g, const DmaTile &t, int m0, int j0, int it)
{
    constexpr int LPP = 2 * AT, PXI = 64 / LPP;
    const int px = it * PXI + s.lane / LPP;
    const int row = t.r0 + s.rg * 16 + (px & 15), m = m0 + (s.lane % LPP) * 8;
    int x = t.x0 + s.cg * BT + j0 + (px >> 4), orow = row;
    bool ok = row < g.rows && m < g.out_CH;
    if (MODE == DM_BWD2) {
        const int n = (int)pc_udiv((uint32_t)row, g.mg_H), y = 2 * (row - n * g.H) + CLS / 2;
        x = 2 * x + CLS % 2;
        orow = n * g.out_H + y;
        ok = ok && y < g.out_H;
    }
    ok = ok && x < g.out_W;
    return ok ? (uint32_t)(orow * g.out_W + x) * (uint32_t)(g.out_CH * 2) + (uint32_t)(m * 2) : DM_OOB;
}

// ahead: the mask elements of the tile (BT <= 4), or null
template <int MODE, int AT, int BT, int CLS, int ACT>
__device__ __forceinline__ void dm_store(const DmaWave &s, const DmaArgs &g, const DmaTile &t, int m0,
                                         const f32x4 (&acc)[AT][MODE == DM_BWD2 ? 4 * BT : BT], unsigned char *stg,
                                         __amdgpu_buffer_rsrc_t osrc, __amdgpu_buffer_rsrc_t msrc, const v4u32 *ahead = nullptr)
{
    constexpr int LPP = 2 * AT, PXI = 64 / LPP, PITCH = 32 * AT + 16;     // lanes per pixel, pixels per store, bytes per pixel in LDS
#pragma unroll
    for (int j0 = 0; j0 < BT; j0 += 4) {
        constexpr int FULL = BT < 4 ? BT : 4;
        const int NC = BT - j0 < FULL ? BT - j0 : FULL;        // columns of this pass
        v4u32 mk[FULL * 16 / PXI];
        uint32_t off[FULL * 16 / PXI];
#pragma unroll
        for (int it = 0; it < NC * 16 / PXI; ++it) {
            off[it] = dm_out_offset<MODE, AT, BT, CLS>(s, g, t, m0, j0, it);
            if (ACT == PC_ACT_RELU_MASK) mk[it] = ahead ? ahead[it] : __builtin_amdgcn_raw_buffer_load_b128(msrc, (int)off[it], 0, 0);
        }
#pragma unroll
        for (int j = 0; j < NC; ++j)
#pragma unroll
            for (int e = 0; e < AT / 2; ++e) {     // 8 of the lane's 4 * AT channels
                v4u32 pv;
#pragma unroll
                for (int u = 0; u < 4; ++u) pv[u] = pc_pack_bf16x2(acc[e * 2 + (u >> 1)][CLS * BT + j0 + j][(u & 1) * 2], acc[e * 2 + (u >> 1)][CLS * BT + j0 + j][(u & 1) * 2 + 1]);
                *reinterpret_cast<v4u32 *>(stg + (j * 16 + (s.lane & 15)) * PITCH + (s.lane >> 4) * (8 * AT) + e * 16) = pv;
            }
#pragma unroll
        for (int it = 0; it < NC * 16 / PXI; ++it) {
            v4u32 pv = *reinterpret_cast<const v4u32 *>(stg + (it * PXI + s.lane / LPP) * PITCH + (s.lane % LPP) * 16);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (ACT == PC_ACT_RELU) pv[u] = pc_relu_bf16x2(pv[u]);
                if (ACT == PC_ACT_RELU_MASK) pv[u] = pc_mask_bf16x2(pv[u], mk[it][u]);
            }
            __builtin_amdgcn_raw_buffer_store_b128(pv, osrc, (int)off[it], 0, 0);
        }
    }
}

template <int AT, int BT> __device__ __forceinline__ void dm_zero(f32x4 (&acc)[AT][BT])
{
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
        for (int j = 0; j < BT; ++j) acc[a][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// One tile of BT columns per wavefront, one buffer. fresh: nothing has used LDS yet.
template <int AT, int BT, int ACT>
__device__ __forceinline__ void dm_one_tile(DmaWave &s, const DmaArgs &g, const DmaGeo &q, unsigned char *lds, __amdgpu_buffer_rsrc_t osrc,
                                            __amdgpu_buffer_rsrc_t msrc, const DmaTile &t, bool &fresh)
{
    dm_offsets<DM_S1, 0>(s, g, q, t);
    const unsigned char *pa = lds + s.lane * 16;
    int rows[3];
    dm_lane_rows<DM_S1, BT>(s, g, q, t, rows);
    const DmaRows pb = dm_rows(lds + AT * (DM_A_BYTES / 4), rows);
    f32x4 acc[AT][BT];
    dm_zero<AT, BT>(acc);
    for (int ch = 0; ch < g.nch; ++ch) {
        if (!fresh) asm volatile("s_barrier" ::: "memory");      // every wavefront has read what the loads replace
        fresh = false;
        __builtin_amdgcn_s_setprio(3);
        int w = s.w;       // (hidden from the compiler here and below: it would compute all scalar offsets ahead and spill them)
        asm volatile("" : "+s"(w));
        dm_issue_weights<DM_S1, AT, AT>(s, g, w, t.mt, ch, 0);
        dm_issue_input<0>(s, g, w, q.nB, ch, AT * (DM_A_BYTES / 4));
        __builtin_amdgcn_s_setprio(0);
        dm_wait_barrier<0>();
        dm_chunk<DM_S1, AT, BT, AT>(acc, pa, pb);
    }
    __builtin_amdgcn_s_setprio(3);
    asm volatile("s_barrier" ::: "memory");
    dm_store<DM_S1, AT, BT, 0, ACT>(s, g, t, t.mt * 64, acc, lds + s.w * (64 * DM_STG), osrc, msrc);
}

// AT = 2: layers of up to 32 output channels. Half the weights and matrix instructions of a tile of 64 channels, of which half would be zeros
// (us: 61 x 199 x 198, 32 -> 16 79.9 -> 55.3; 103 x 178 x 180, 8 -> 24 82.0 -> 65.4; 66 x 50 x 47, 96 -> 16 17.8 -> 11.8; 60 layers, the kernel chosen
// before and the fastest of these forms: 1.19 on average).
template <int BT, int ACT, int AT>
__global__ void __launch_bounds__(256, 2)
pc_mfma_conv_dma_kernel(const uint16_t *__restrict__ in, uint16_t *__restrict__ out, const uint16_t *__restrict__ wz, DmaArgs g)
{
    extern __shared__ __align__(16) unsigned char lds[];
    DmaWave s;
    s.lane = threadIdx.x & 63;
    s.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    s.cg = s.w & ((1 << g.lgCG) - 1);
    s.rg = s.w >> g.lgCG;
    const int G = gridDim.x, b = blockIdx.x;
    // Workgroups go to the XCDs round robin, and to a CU a second time when each has one: neighbours in the tile order share an XCD, and
    // what does not fill a round has a CU each.
    const int vb = (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
    const int vl = (g.last & 7) == 0 ? (b & 7) * (g.last >> 3) + (b >> 3) : b;
    s.xs = dm_rsrc(in, g.in_bytes);
    s.ws = dm_rsrc(wz, g.wz_bytes);
    s.a_voff = dm_weight_offset<AT>(g, s.lane);
    const __amdgpu_buffer_rsrc_t osrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, g.out_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t msrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(ACT == PC_ACT_RELU_MASK ? g.act_mask : out), 0, g.out_bytes, 0x00020000);
    const int ntile = g.rounds + (b < g.last);
    bool fresh = true;
    for (int k = 0; k < ntile; ++k)
        dm_one_tile<AT, BT, ACT>(s, g, g.geo[0], lds, osrc, msrc, dm_tile<BT>(g, k < g.rounds ? k * G + vb : g.rounds * G + vl, 0), fresh);
    if constexpr (BT == 8 || BT == 4) {
        const int p0 = (g.rounds * G + g.last) << g.lgP;
        for (int u = (b - g.last + 2 * G) % G; u < g.pieces; u += G) {
            const DmaTile t = dm_tile<BT>(g, p0 + u, g.lgP);
            if (g.lgP == 1) dm_one_tile<AT, BT / 2, ACT>(s, g, g.geo[1], lds, osrc, msrc, t, fresh);
            else if constexpr (BT == 8) dm_one_tile<AT, 2, ACT>(s, g, g.geo[2], lds, osrc, msrc, t, fresh);
        }
    }
}

// One workgroup of 8 wavefronts per CU: four multiply, four issue the direct loads of the chunks ahead, up to NBUF - 1 of them (a
// wavefront issues in order, and 48 to 77 KiB of loads take 800 to 1200 cycles to be accepted: with the loads in the multiplying
// wavefronts a chunk of the smaller tiles took twice its matrix instructions). AT = 2: the wavefronts are two halves of the
// channels x two groups of pixels, tiles of 64 x 128 (BT = 4) and 64 x 64 (BT = 2).
// What bounds it: a chunk of 64 x 256, 128 and 64 pixels takes 1.15, 0.64 and 0.39 us for 0.96, 0.48 and 0.24 us of matrix
// instructions; below 64 x 128 the direct loads (48 KiB a chunk, of them 36 KiB weights that all row tiles load again). With a launch and
// the first loads (2 us) and last stores around them, in a graph, 128 images (us, the fastest kernel with operands in registers -> here): 16 x 16
// 128 -> 128 11.5 -> 9.7, 8 x 8 256 -> 256 11.6 -> 9.3, 4 x 4 512 -> 512 11.9 -> 10.6, 4 x 4 256 -> 512 8.5 -> 7.2; 64 images 7 x 7
// 512 -> 512 16.9 -> 14.9; one image 56 x 56 256 -> 256 7.9 -> 6.9.
// Stride 2, backward-data: the same nine taps per chunk and fewer staged columns, 128 images 8 x 8 256 -> 512 16.8 -> 10.7, 64 images
// 14 x 14 256 -> 512 17.5 -> 11.7, 56 x 56 128 -> 128 25.7 -> 22.6 (its bytes). Forward: 2 * BT + 1 fragments per row and four staged
// pixels per output pixel make LDS the bound, 0.9 us a chunk of 64 x 128 for 0.48 of matrix instructions (1.5 where the input comes from
// memory): 64 images 14 x 14 256 -> 512 12.5 -> 11.9, 128 images 16 x 16 128 -> 256 12.2 -> 8.4; of large maps with few channels
// tiles of 128 channels read less (pc_mfma_conv_ring_kernel below).
template <int MODE, int AT, int BT, int NBUF, int ACT>
__global__ void __launch_bounds__(512, 2)
pc_mfma_conv_solo_kernel(const uint16_t *__restrict__ in, uint16_t *__restrict__ out, const uint16_t *__restrict__ wz, DmaArgs g)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NBW = NBUF == 3 ? dm_nbw(BT) : 0;
    DmaWave s;
    s.lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    s.w = wave & 3;
    const int pw = AT == 2 ? s.w >> 1 : s.w;
    s.cg = pw & ((1 << g.lgCG) - 1);
    s.rg = pw >> g.lgCG;
    const int G = gridDim.x, b = blockIdx.x;
    const int vb = (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
    const int vl = (g.last & 7) == 0 ? (b & 7) * (g.last >> 3) + (b >> 3) : b;
    const int ntile = g.rounds + (b < g.last), nch = g.nch;
    auto tile_at = [&](int k) { return dm_tile<BT>(g, k < g.rounds ? k * G + vb : g.rounds * G + vl, 0); };
    const DmaGeo &q = g.geo[0];
    const int buf_bytes = (int)g.buf_bytes;

    if (wave >= 4) {
        s.xs = dm_rsrc(in, g.in_bytes);
        s.ws = dm_rsrc(wz, g.wz_bytes);
        s.a_voff = dm_weight_offset<AT>(g, s.lane);
        const int nB = q.nB, chunks = ntile * nch;
        DmaTile t = tile_at(0);
        dm_issue_weights<MODE, AT, 4>(s, g, s.w, t.mt, 0, 0);      // (on their way while the offsets are made)
        dm_offsets<MODE, NBW, true>(s, g, q, t, DM_A_BYTES);
        int k = 0, ch = 0, at = 0, done = 0;       // cursor: tile, chunk, buffer; chunks issued
        auto next = [&]() {
            int w = s.w;
            asm volatile("" : "+s"(w));
            if (done) {
                dm_issue_weights<MODE, AT, 4>(s, g, w, t.mt, ch, at);
                dm_issue_input<NBW>(s, g, w, nB, ch, at + DM_A_BYTES);
            }
            at = at + buf_bytes == NBUF * buf_bytes ? 0 : at + buf_bytes;
            ++done;
            if (++ch == nch) {
                ch = 0;
                if (++k < ntile) {
                    t = tile_at(k);
                    dm_offsets<MODE, NBW>(s, g, q, t);
                }
            }
        };
        for (int i = 0; i < NBUF - 1; ++i)
            if (done < chunks) next();
        int left = nch;
        for (int i = 0; i < chunks; ++i) {
            // chunk i is complete, and the buffer of chunk i - 1 is free
            if (NBUF == 3 && done > i + 1) dm_wait_barrier<9 + NBW>();
            else dm_wait_barrier<0>();
            if (done < chunks) next();
            if (--left == 0) {
                left = nch;
                asm volatile("s_barrier" ::: "memory");      // (the tile's sums leave through the buffer of its last chunk)
            }
        }
        return;
    }
    const __amdgpu_buffer_rsrc_t osrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, g.out_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t msrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(ACT == PC_ACT_RELU_MASK ? g.act_mask : out), 0, g.out_bytes, 0x00020000);
    const int half = AT == 2 ? s.w & 1 : 0;
    // Weights come from the last cache or from memory after other layers' work, chunk by chunk, each with that latency and two chunks ahead
    // at most. These wavefronts wait for the first chunk anyway: together the workgroups of an XCD that share a row tile touch every
    // 128-byte line of its weights once, so that the chunks come from L2. (In a step of many layers, 128 images 4 x 4 512 -> 512
    // 15.5 -> 12.2 us, 64 images 7 x 7 512 -> 512 18.2 -> 16.7, stride 2 8 x 8 256 -> 512 15.2 -> 13.6 forward, 16.2 -> 13.2
    // backward-data. At stride 1 with more input than weights an XCD reads all row tiles and few workgroups share each: 0.2
    // to 0.5 us slower, not done. The input ahead: 1 us slower.)
    uint32_t touched[4];
    const int lines = 18 * g.KS * 8, part = g.share ? (lines + g.share - 1) / g.share : 0, mt0 = tile_at(0).mt;
    const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wz), 0, g.wz_bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int l = i * 256 + (int)threadIdx.x, line = (b >> 3) / g.apart * part + l;
        touched[i] = __builtin_amdgcn_raw_buffer_load_b32(wsrc, (int)(l < part && line < lines ? (uint32_t)((mt0 * lines + line) * 128) : DM_OOB), 0, 0);
    }
    int at = 0;
    for (int k = 0; k < ntile; ++k) {
        const DmaTile t = tile_at(k);
        const unsigned char *pa = lds + s.lane * 16 + half * 2048;
        int rows[3];
        dm_lane_rows<MODE, BT>(s, g, q, t, rows);
        v4u32 mk[BT * AT / 2];
        if (ACT == PC_ACT_RELU_MASK) {
#pragma unroll
            for (int i = 0; i < BT * AT / 2; ++i)
                mk[i] = __builtin_amdgcn_raw_buffer_load_b128(msrc, (int)dm_out_offset<MODE, AT, BT, 0>(s, g, t, t.mt * 64 + half * 32, 0, i), 0, 0);
        }
        f32x4 acc[AT][MODE == DM_BWD2 ? 4 * BT : BT];
        dm_zero(acc);
        int used = 0;
        for (int ch = 0; ch < nch; ++ch) {
            asm volatile("s_barrier" ::: "memory");
            dm_chunk<MODE, AT, BT>(acc, pa + at, dm_rows(lds + DM_A_BYTES + at, rows));
            used = at;
            at = at + buf_bytes == NBUF * buf_bytes ? 0 : at + buf_bytes;
        }
        asm volatile("s_barrier" ::: "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" :: "v"(touched[i]));      // (no earlier: the wait for them stands here)
        unsigned char *stg = lds + used + s.w * (64 * (32 * AT + 16));
        dm_store<MODE, AT, BT, 0, ACT>(s, g, t, t.mt * 64 + half * 32, acc, stg, osrc, msrc, ACT == PC_ACT_RELU_MASK ? mk : nullptr);
        if constexpr (MODE == DM_BWD2) {
            dm_store<MODE, AT, BT, 1, ACT>(s, g, t, t.mt * 64 + half * 32, acc, stg, osrc, msrc);
            dm_store<MODE, AT, BT, 2, ACT>(s, g, t, t.mt * 64 + half * 32, acc, stg, osrc, msrc);
            dm_store<MODE, AT, BT, 3, ACT>(s, g, t, t.mt * 64 + half * 32, acc, stg, osrc, msrc);
        }
    }
}

// Layers of up to 64 input and 16 * AT output channels, 64 and 32, whose weights stay in LDS: a workgroup of 8 wavefronts per CU, four multiply, four
// load tiles of 16 * AT channels x 64 * BT pixels a chunk of 32 channels at a time into three buffers. A tile's sums leave through LDS of their
// own, so the loads of the next tiles go on meanwhile. What bounds these layers is memory: with the kernels above a chunk loads 36 KiB of
// weights again beside 20 to 40 KiB of input, and loads, products and stores of a CU's two workgroups overlap in part. us, the fastest of the
// others -> here: 32 x 224 x 224, 64 -> 64 114 -> 99 forward and backward (4.1 TB/s; in a training step 124 -> 95 and, with the mask, 149 -> 130), 32 x
// 112 x 112 31.5 -> 29.3, one 224 x 224 image 7.6 -> 7.0, 61 x 199 x 198, 32 -> 16 53.5 -> 48.5; 64 x 56 x 56 (three tiles a CU and 16 left) 18.5
// -> 19.5: by the estimate.
template <int AT, int BT, int NBW, int ACT>
__global__ void __launch_bounds__(512, 2)
pc_mfma_conv_keep_kernel(const uint16_t *__restrict__ in, uint16_t *__restrict__ out, const uint16_t *__restrict__ wz, DmaArgs g)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int WB = AT * (DM_A_BYTES / 4), BUF = 4 * NBW * 1024;      // bytes of a chunk's weights and of an input buffer
    DmaWave s;
    s.lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    s.w = wave & 3;
    s.cg = s.w & ((1 << g.lgCG) - 1);
    s.rg = s.w >> g.lgCG;
    const int G = gridDim.x, b = blockIdx.x;
    const int vb = (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
    const int vl = (g.last & 7) == 0 ? (b & 7) * (g.last >> 3) + (b >> 3) : b;
    const int ntile = g.rounds + (b < g.last), nch = g.nch, x0 = nch * WB;
    auto tile_at = [&](int k) { return dm_tile<BT>(g, k < g.rounds ? k * G + vb : g.rounds * G + vl, 0); };
    const DmaGeo &q = g.geo[0];

    if (wave >= 4) {
        s.xs = dm_rsrc(in, g.in_bytes);
        s.ws = dm_rsrc(wz, g.wz_bytes);
        s.a_voff = dm_weight_offset<AT>(g, s.lane);
        const int chunks = ntile * nch;
        DmaTile t = tile_at(0);
        dm_issue_weights<DM_S1, AT, AT>(s, g, s.w, 0, 0, 0);
        dm_offsets<DM_S1, NBW, true>(s, g, q, t, x0);
        int k = 0, ch = 0, at = x0, done = 0;      // cursor: tile, chunk, buffer; chunks issued
        auto next = [&]() {
            int w = s.w;
            asm volatile("" : "+s"(w));
            if (done) dm_issue_input<NBW>(s, g, w, 0, ch, at);
            at = at == x0 + 2 * BUF ? x0 : at + BUF;
            ++done;
            if (++ch == nch) {
                ch = 0;
                if (++k < ntile) {
                    t = tile_at(k);
                    dm_offsets<DM_S1, NBW>(s, g, q, t);
                }
            }
        };
        next();
        if (nch == 2) dm_issue_weights<DM_S1, AT, AT>(s, g, s.w, 0, 1, WB);
        if (done < chunks) next();
        for (int i = 0; i < chunks; ++i) {
            // chunk i is complete, and the buffer of chunk i - 1 is free
            if (i == 0 && nch == 2) dm_wait_barrier<(AT == 4 ? 9 : 4) + NBW>();
            else if (done > i + 1) dm_wait_barrier<NBW>();
            else dm_wait_barrier<0>();
            if (done < chunks) next();
        }
        return;
    }
    constexpr int LPP = 2 * AT, PXI = 64 / LPP, IT = 16 / PXI, PITCH = AT == 4 ? 128 : 80;   // lanes per pixel, pixels per store, stores per column, bytes per pixel in LDS
    const __amdgpu_buffer_rsrc_t osrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, g.out_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t msrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(ACT == PC_ACT_RELU_MASK ? g.act_mask : out), 0, g.out_bytes, 0x00020000);
    const int pix = g.out_CH * 2;
    unsigned char *stg = lds + x0 + 3 * BUF + s.w * (2 * 16 * PITCH);
    // (rows of 128 bytes: their 16-byte pieces are stored in turned order, or all pixels' would stand in the same banks)
    auto piece = [&](int px, int i) { return AT == 4 ? i ^ (px & 7) : i; };
    int at = x0;
    for (int k = 0; k < ntile; ++k) {
        const DmaTile t = tile_at(k);
        const unsigned char *pa = lds + s.lane * 16;
        int rows[3];
        dm_lane_rows<DM_S1, BT>(s, g, q, t, rows);
        uint32_t off[IT];                          // of this lane's pixels in column 0 of the map
        v4u32 mk[BT][IT];
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int row = t.r0 + s.rg * 16 + i * PXI + s.lane / LPP, m = (s.lane % LPP) * 8;
            off[i] = row < g.rows && m < g.out_CH ? (uint32_t)(row * g.out_W) * (uint32_t)pix + (uint32_t)(m * 2) : DM_OOB;
        }
        const int xw = t.x0 + s.cg * BT;
        if (ACT == PC_ACT_RELU_MASK) {
#pragma unroll
            for (int j = 0; j < BT; ++j)
#pragma unroll
                for (int i = 0; i < IT; ++i) mk[j][i] = __builtin_amdgcn_raw_buffer_load_b128(msrc, (int)(xw + j < g.out_W ? off[i] : DM_OOB), xw + j < g.out_W ? (xw + j) * pix : 0, 0);
        }
        f32x4 acc[AT][BT];
        dm_zero<AT, BT>(acc);
        for (int ch = 0; ch < nch; ++ch) {
            asm volatile("s_barrier" ::: "memory");
            dm_chunk<DM_S1, AT, BT, AT>(acc, pa + ch * WB, dm_rows(lds + at, rows));
            at = at == x0 + 2 * BUF ? x0 : at + BUF;
        }
#pragma unroll
        for (int j0 = 0; j0 < BT; j0 += 2) {
            const int NC = BT - j0 < 2 ? BT - j0 : 2;
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int e = 0; e < AT / 2; ++e) {     // 8 of the lane's 4 * AT channels
                    v4u32 pv;
#pragma unroll
                    for (int u = 0; u < 4; ++u) pv[u] = pc_pack_bf16x2(acc[e * 2 + (u >> 1)][j0 + j][(u & 1) * 2], acc[e * 2 + (u >> 1)][j0 + j][(u & 1) * 2 + 1]);
                    const int px = s.lane & 15;
                    *reinterpret_cast<v4u32 *>(stg + (j * 16 + px) * PITCH + piece(px, (s.lane >> 4) * (AT / 2) + e) * 16) = pv;
                }
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int i = 0; i < IT; ++i) {
                    const int px = i * PXI + s.lane / LPP, x = xw + j0 + j;
                    v4u32 pv = *reinterpret_cast<const v4u32 *>(stg + (j * 16 + px) * PITCH + piece(px, s.lane % LPP) * 16);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (ACT == PC_ACT_RELU) pv[u] = pc_relu_bf16x2(pv[u]);
                        if (ACT == PC_ACT_RELU_MASK) pv[u] = pc_mask_bf16x2(pv[u], mk[j0 + j][i][u]);
                    }
                    __builtin_amdgcn_raw_buffer_store_b128(pv, osrc, (int)(x < g.out_W ? off[i] : DM_OOB), x < g.out_W ? x * pix : 0, 0);
                }
        }
    }
}

// The stride-2 forward pass in tiles of 128 output channels x 128 pixels, 8 wavefronts, four of them loading: two input buffers, and the
// weights, a row of taps at a time, in a ring of three places (72 + 88 KiB: whole chunks of both would not fit twice). A wavefront
// multiplies 64 channels x 64 pixels, so that a chunk reads 252 KiB of LDS where two tiles of 64 channels read 360, and an input
// tile is loaded once for 128 channels. 1.56 us a chunk (0.96 of matrix instructions; LDS 1.2 and a wait at every row). 64 images, us,
// with the best of the other kernels -> here: 56 x 56 64 -> 128 16.2 -> 14.0, 128 -> 128 25.6 -> 23.2, 28 x 28 128 -> 256 12.8 -> 11.6; 11
// images 52 x 53 232 -> 480 27.3 -> 21.3; fastest of all on 9 of the 148 drawn layers in
// profiles/plan_timings_bf16.csv.
#define DR_B 44                      // direct loads of an input tile: 6 and 5 per wavefront in the first two steps of a chunk
#define DR_W (2 * DR_B * 1024)       // where the ring begins
#define DR_SLOT (24 * 1024)

template <int ACT>
__global__ void __launch_bounds__(512, 2)
pc_mfma_conv_ring_kernel(const uint16_t *__restrict__ in, uint16_t *__restrict__ out, const uint16_t *__restrict__ wz, DmaArgs g)
{
    extern __shared__ __align__(16) unsigned char lds[];
    DmaWave s;
    s.lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    s.w = wave & 3;
    const int half = s.w & 1;
    s.cg = (s.w >> 1) & ((1 << g.lgCG) - 1);
    s.rg = (s.w >> 1) >> g.lgCG;
    const int G = gridDim.x, b = blockIdx.x;
    const int vb = (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
    const int vl = (g.last & 7) == 0 ? (b & 7) * (g.last >> 3) + (b >> 3) : b;
    const int ntile = g.rounds + (b < g.last), nch = g.nch;
    auto tile_at = [&](int k) { return dm_tile<4>(g, k < g.rounds ? k * G + vb : g.rounds * G + vl, 0); };
    const DmaGeo &q = g.geo[0];

    if (wave >= 4) {
        s.xs = dm_rsrc(in, g.in_bytes);
        s.ws = dm_rsrc(wz, g.wz_bytes);
        s.a_voff = dm_weight_offset<4>(g, s.lane);
        const int steps = 3 * nch * ntile;
        DmaTile tw = tile_at(0);
        int kw = 0, chw = 0, rw = 0, slot = 0, wdone = 0;      // weights: tile, chunk, row of taps, place, rows issued
        auto weights = [&]() {
            int w = s.w;
            asm volatile("" : "+s"(w));
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    dm_load(s.ws, s.a_voff, (((tw.mt * 2 + h) * 18 + rw * 3 + t) * g.KS + chw * 2) * 1024 + w * 64, DR_W + slot + (t * 8 + h * 4 + w) * 1024);
            slot = slot == 2 * DR_SLOT ? 0 : slot + DR_SLOT;
            ++wdone;
            if (++rw == 3) {
                rw = 0;
                if (++chw == nch) {
                    chw = 0;
                    if (++kw < ntile) tw = tile_at(kw);
                }
            }
        };
        DmaTile tx = tw;
        int kx = 0, chx = 0, at = 0;
        weights();                                // (on their way while the offsets are made)
        dm_offsets<DM_FWD2, 11, true>(s, g, q, tx, 0);
        bool ask = false;                         // (the first chunk: on its way)
        auto input = [&](auto part) {          // 0: the first 6 loads, 1: the other 5, and on to the next chunk
            const bool cut = chx == nch - 1 && (g.in_CH & (DM_KC - 1));
            const uint32_t parts = (uint32_t)(g.in_CH & (DM_KC - 1)) >> 3;
#pragma unroll
            for (int i = decltype(part)::value ? 6 : 0; i < (decltype(part)::value ? 11 : 6); ++i) {
                uint32_t vo = s.voff[i];
                if (cut) vo = ((s.part >> (2 * i)) & 3u) >= parts ? DM_OOB : vo;
                if (ask) dm_load(s.xs, (int)vo, chx * (DM_KC * 2), at + (s.w + 4 * i) * 1024);
            }
            if (decltype(part)::value) {
                at = DR_B * 1024 - at;
                if (++chx == nch) {
                    chx = 0;
                    if (++kx < ntile) {
                        tx = tile_at(kx);
                        dm_offsets<DM_FWD2, 11>(s, g, q, tx);
                    }
                }
            }
        };
        using first = std::integral_constant<int, 0>;
        using rest = std::integral_constant<int, 1>;
        input(first());
        input(rest());
        ask = true;
        weights();
        int newer = 6, r = 0, left = nch;         // newer: loads of the last step, which nothing waits for yet
        for (int i = 0; i < steps; ++i) {
            if (newer == 12) dm_wait_barrier<12>();
            else if (newer == 11) dm_wait_barrier<11>();
            else if (newer == 6) dm_wait_barrier<6>();
            else dm_wait_barrier<0>();
            newer = 0;
            if (wdone < steps) { weights(); newer = 6; }
            if (r < 2 && kx < ntile) {
                if (r == 0) { input(first()); newer += 6; }
                else { input(rest()); newer += 5; }
            }
            if (++r == 3) {
                r = 0;
                if (--left == 0) {
                    left = nch;
                    asm volatile("s_barrier" ::: "memory");      // (the tile's sums leave through the input buffer of its last chunk)
                }
            }
        }
        return;
    }
    const __amdgpu_buffer_rsrc_t osrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, g.out_bytes, 0x00020000);
    int at = 0, slot = 0;
    for (int k = 0; k < ntile; ++k) {
        const DmaTile t = tile_at(k);
        const unsigned char *pa = lds + DR_W + s.lane * 16 + half * 4096;
        int rows[3];
        dm_lane_rows<DM_FWD2, 4>(s, g, q, t, rows);
        f32x4 acc[4][4];
        dm_zero(acc);
        int used = 0;
        for (int ch = 0; ch < nch; ++ch) {
            bf16x8 aq[2][4], bq[9];
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                asm volatile("s_barrier" ::: "memory");
                const unsigned char *pw = pa + slot, *pr = lds + at + rows[0];
                slot = slot == 2 * DR_SLOT ? 0 : slot + DR_SLOT;
#pragma unroll
                for (int a = 0; a < 4; ++a) aq[0][a] = *reinterpret_cast<const bf16x8 *>(pw + a * 1024);
                if (r == 0) {
#pragma unroll
                    for (int c = 0; c < 9; ++c) bq[c] = *reinterpret_cast<const bf16x8 *>(pr + c * 64);
                }
                const unsigned char *pn = lds + at + rows[r == 0 ? 1 : 2];
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const bool refill = u == 2 && r < 2;       // (the input is there: the next row's fragments, before its weights)
                    auto read = [&](int c) { bq[c] = *reinterpret_cast<const bf16x8 *>(pn + c * 64); };
                    if (refill) { read(0); read(1); }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (u < 2) aq[(u + 1) & 1][j] = *reinterpret_cast<const bf16x8 *>(pw + ((u + 1) * 8 + j) * 1024);
#pragma unroll
                        for (int a = 0; a < 4; ++a) acc[a][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq[u & 1][a], bq[2 * j + u], acc[a][j], 0, 0, 0);
                        if (refill) {
                            read(2 * j + 2);
                            if (j < 3) read(2 * j + 3);
                        }
                    }
                    if (refill) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (u < 2) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                        if (refill && j < 3) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        else if (refill) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            used = at;
            at = DR_B * 1024 - at;
        }
        asm volatile("s_barrier" ::: "memory");
        dm_store<DM_FWD2, 4, 4, 0, ACT>(s, g, t, t.mt * 128 + half * 64, acc, lds + used + s.w * (64 * DM_STG), osrc, osrc);
    }
}

// ---- plan and launch
// Constants of the time estimate (us) of a tile: a chunk, each direct load of its input, the tile's end; of the launch: its start, and a
// factor for the time of its bytes
struct DmaTimes { double chunk, load, tile, start, bytes; };
#define DM_KEEP_NBW 6                // direct loads of a chunk per loading wavefront where the weights stay in LDS
struct DmaCand { int code, mode, at, bt, nbuf; DmaTimes solo; };       // nbuf 1: two workgroups per CU; 4: the weights stay in LDS beside three
static const DmaCand kDma[] = {
    {40, DM_S1, 4, 8, 1, {0, 0, 0, 2.93, 1.07}}, {41, DM_S1, 4, 4, 1, {0, 0, 0, 2.73, 1.04}}, {42, DM_S1, 4, 7, 1, {0, 0, 0, 2.90, 0.89}},
    {43, DM_S1, 2, 4, 3, {0.639, 0, 0.530, 2.72, 0.70}}, {45, DM_S1, 4, 4, 2, {1.152, 0.0009, 0.80, 2.95, 0.85}}, {46, DM_S1, 2, 2, 3, {0.368, 0.0037, 0.487, 2.65, 0.69}},
    {47, DM_FWD2, 2, 4, 2, {0.976, 0, 1.296, 2.7, 0.78}}, {49, DM_FWD2, 8, 4, 2, {1.5, 0, 1.8, 2.6, 0.7}}, {48, DM_FWD2, 2, 2, 2, {0.716, 0, 1.275, 2.5, 0.78}},
    {50, DM_S1, 4, 4, 4, {0, 0, 0, 0, 0}},
    {37, DM_BWD2, 2, 4, 3, {0.504, 0.0087, 1.829, 3.1, 0.62}}, {38, DM_BWD2, 2, 2, 3, {0.348, 0.0082, 1.210, 2.9, 0.50}}};
constexpr int kNumDma = sizeof(kDma) / sizeof(kDma[0]);

// Fills the plan for a kernel and 1 << lgCG wavefronts side by side; false when it does not fit.
static bool plan_dma(const MfmaArgs &g, bool flip, const DmaCand &cand, int lgCG, DmaArgs *out, size_t *lds, int *grid, double *est, int num_cu)
{
    DmaArgs t;
    memset(&t, 0, sizeof(t));
    t.N = g.N; t.H = g.GH; t.W = g.GW; t.in_CH = g.in_CH; t.out_CH = g.out_CH;
    t.in_H = g.in_H; t.in_W = g.in_W; t.out_H = g.out_H; t.out_W = g.out_W;
    t.KS = g.KS; t.nch = (g.in_CH + DM_KC - 1) / DM_KC; t.flip = flip;
    t.lgCG = lgCG;
    const bool keep = cand.nbuf == 4;
    if (keep && (g.in_CH > 64 || g.out_CH > 64)) return false;
    const bool narrow = (cand.nbuf == 1 || keep) && g.out_CH <= 32;
    const int lgPG = cand.at == 4 ? 2 : 1, rows_m = cand.at == 8 ? 128 : 64;       // groups of pixels among the wavefronts (log2)
    if (lgCG > lgPG) return false;
    t.TR = 16 << (lgPG - lgCG);
    const int64_t rows = (int64_t)g.N * t.H;
    if ((rows + g.N + 2 * t.TR) * (t.H + 1) >= ((int64_t)1 << 32) || rows >= (1 << 24)) return false;   // multiply-high divisions stay exact
    t.rows = (int)rows;
    // image boundaries inside a tile (tiles start at multiples of TR)
    int cross = t.H % t.TR == 0 ? 0 : t.TR % t.H == 0 ? t.TR / t.H - 1 : (t.TR - 1 + t.H - 1) / t.H;
    if (cross > g.N - 1) cross = g.N - 1;
    t.nrow = cand.mode == DM_S1 ? t.TR + 2 : t.TR + 1 + cross;
    const int staged = cand.mode == DM_FWD2 ? 2 * t.nrow : t.nrow;
    const int most = cand.at == 8 ? DR_B : 4 * (keep ? DM_KEEP_NBW : cand.nbuf == 3 ? dm_nbw(cand.bt) : DM_NB);
    for (int l = 0; l < 3; ++l) {
        DmaGeo &q = t.geo[l];
        const int bt = cand.bt >> l, tc = bt << lgCG;
        q.IW = cand.mode == DM_S1 ? tc + 2 : cand.mode == DM_FWD2 ? 2 * tc + 1 : tc + 1;
        for (int pad = 2; pad >= 1; --pad) {       // (one element where two do not fit)
            q.EPR = (DM_KC / 8) * q.IW + pad;
            int elements = staged * q.EPR;
            if (cand.mode == DM_S1) {              // zeros: 256 bytes and the fragments of a row
                elements = (elements + 15) / 16 * 16;
                q.zero = elements * 16;
                elements += 16 + 4 * (bt + 2);
            }
            q.nB = (elements + 63) / 64;
            if (q.nB <= most && (keep || cand.at == 8 || ((narrow ? DM_A_BYTES / 2 : DM_A_BYTES) + q.nB * 1024) * (cand.nbuf == 3 ? 1 : cand.nbuf) <= DM_LDS_MAX / (cand.nbuf == 1 ? 2 : 1))) break;
        }
        q.mg_EPR = pc_udiv_magic(q.EPR);
    }
    const int nB = t.geo[0].nB, TC = cand.bt << lgCG;
    if (nB > most) return false;
    t.buf_bytes = cand.at == 8 ? DM_LDS_MAX / 2 : (narrow ? DM_A_BYTES / 2 : DM_A_BYTES) + (uint32_t)(cand.nbuf == 3 ? 4 * dm_nbw(cand.bt) : nB) * 1024;
    if (keep) {
        t.buf_bytes = 4 * DM_KEEP_NBW * 1024;
        *lds = t.nch * (size_t)(narrow ? DM_A_BYTES / 2 : DM_A_BYTES) + 3 * (size_t)t.buf_bytes + 4 * 2 * 16 * (narrow ? 80 : 128);
        if (*lds > (size_t)DM_LDS_MAX) return false;
    }
    if (!keep && narrow && t.buf_bytes < 4 * 64 * DM_STG) t.buf_bytes = 4 * 64 * DM_STG;      // (the tile leaves through it)
    if (!keep) *lds = (size_t)t.buf_bytes * cand.nbuf;
    if (!keep && *lds > (size_t)DM_LDS_MAX / (cand.nbuf == 1 ? 2 : 1)) return false;
    t.tiles_x = (t.W + TC - 1) / TC;
    const int64_t p_tiles = (rows + t.TR - 1) / t.TR * t.tiles_x;
    const int m_tiles = (g.out_CH + rows_m - 1) / rows_m;
    const int64_t total = p_tiles * m_tiles;
    const int64_t in_bytes = (int64_t)g.N * g.in_H * g.in_W * g.in_CH * 2, out_bytes = (int64_t)g.N * g.out_H * g.out_W * g.out_CH * 2;
    if (total > (1 << 28) || in_bytes >= ((int64_t)1 << 31) || out_bytes >= ((int64_t)1 << 31)) return false;
    t.in_bytes = (uint32_t)in_bytes; t.out_bytes = (uint32_t)out_bytes;
    t.wz_bytes = (uint32_t)((size_t)((g.out_CH + 127) / 128 * 4) * 9 * t.KS * 1024);
    t.m_fast = in_bytes >= (int64_t)g.out_CH * g.in_CH * 18;     // neighbours share the larger operand
    t.fdiv = t.m_fast ? m_tiles : (int)p_tiles;
    if (total * (t.fdiv > t.tiles_x ? t.fdiv : t.tiles_x) >= ((int64_t)1 << 32)) return false;
    t.mg_fd = pc_udiv_magic(t.fdiv); t.mg_tx = pc_udiv_magic(t.tiles_x);
    t.mg_H = pc_udiv_magic(t.H); t.mg_H1 = pc_udiv_magic(t.H + 1);
    t.act_mask = g.act_mask;
    // Estimated time (us). A round is one tile for each of the workgroups the chip holds, two per CU; a workgroup that has its CU to
    // itself takes its chunks faster. A chunk takes a fixed time and one for its direct loads of the input, a tile an end; the
    // tensors take their bytes (the input with its border, in pieces of 64) at 6 TB/s (7.9 where they come from the last cache, as
    // in a loop over one layer). Constants from 4700 timings of 485 layer shapes at stride 1 (1 to 128 images, 4 x 4 to
    // 224 x 224, 8 to 512 channels, a half of them layers of networks; 5 to 8 % rms) and of 139 at stride 2. On the layers of
    // profiles/plan_timings_bf16.csv the choice, the register and cooperative kernels included, is 1.4 % behind the fastest at stride 1 (both
    // passes), 1.0 % at stride 2 forward and 0.3 % backward, the worst 22 %; on the 540 passes of networks 0.4 %.
    // What does not fill a round of tiles may be cut in halves or quarters, all of it or what a tile per CU leaves: 56 x 56,
    // 256 -> 256, batch 32 is 784 tiles of 8 columns for 512 workgroups; 512 + 256 tiles and 16 cut into 64 quarters
    // take 73 us instead of 81.
    static const DmaTimes kPair[4] = {{2.663, 0.0396, 2.256}, {2.151, 0.0391, 2.288}, {1.605, 0.0194, 1.506}, {0.996, 0.0344, 1.348}};
    static const DmaTimes kOne[4] = {{3.001, 0.0001, 1.680}, {2.519, 0.0000, 1.373}, {1.527, 0.0034, 0.848}, {0.996, 0.0099, 0.638}};
    // Up to 32 output channels: shares of these times, by tile width (660 timings of 220 layers, 4 to 6 % rms).
    // A chunk is half a line of a pixel: where the lines under way exceed the L2s (28 MB; all of them from 60 MB on) the next chunk fetches
    // them again (27 x 96 x 93, 360 -> 8: 81.8 us in tiles of 8 columns, 51.0 in tiles of 4).
    static const DmaTimes kNarrow[3] = {{0.669, 0.444, 0.310, 3.13, 0.833}, {0.614, 0.407, 0.285, 2.86, 0.75}, {0.645, 0.428, 0.299, 2.87, 0.809}};
    const int first = cand.bt == 8 ? 0 : cand.bt == 7 ? 1 : 2;
    auto tile_us = [&](const DmaTimes &c, int l) {
        return narrow ? t.nch * (kNarrow[first].chunk * c.chunk + kNarrow[first].load * c.load * t.geo[l].nB) + kNarrow[first].tile * c.tile : t.nch * (c.chunk + c.load * t.geo[l].nB) + c.tile;
    };
    const int slots = num_cu * (cand.nbuf == 1 ? 2 : 1);
    t.rounds = (int)(total / slots);
    const int left = (int)(total % slots);
    double best = 1e30;
    for (int o = 0; o < 5; ++o) {      // 0: whole tiles; 1, 2: a whole tile per CU and the rest in halves, quarters; 3, 4: all of it
        const int lgP = o == 0 ? 0 : o & 1 ? 1 : 2;
        if (o && (cand.nbuf > 1 || (cand.bt != 8 && !(cand.bt == 4 && lgP == 1)))) continue;
        if ((o == 1 || o == 2) && left <= num_cu) continue;
        const int last = o == 0 ? left : o < 3 ? num_cu : 0, pieces = o == 0 ? 0 : (left - last) << lgP;
        const DmaTimes &pair = cand.nbuf > 1 ? cand.solo : kPair[first], &ppair = kPair[cand.bt == 8 && lgP == 1 ? 2 : 3], &pone = kOne[cand.bt == 8 && lgP == 1 ? 2 : 3];
        double c = (t.rounds + (last > (cand.nbuf > 1 ? 0 : num_cu))) * tile_us(pair, 0);
        if (cand.nbuf == 1 && last > 0 && last <= num_cu) c += tile_us(kOne[first], 0);
        if (pieces && last) c += 0.83 * tile_us(ppair, lgP);
        else if (pieces) c += (pieces / slots + (pieces % slots > num_cu)) * tile_us(ppair, lgP) + (pieces % slots > 0 && pieces % slots <= num_cu ? tile_us(pone, lgP) : 0.0);
        if (c < best) { best = c; t.last = last; t.pieces = pieces; t.lgP = lgP; }
    }
    double in_moved = 2.0 * (double)p_tiles * staged * t.geo[0].IW * (g.in_CH < DM_KC ? DM_KC : g.in_CH);
    if (narrow && !keep && t.nch > 1) {
        const double under_way = (double)(total < slots ? total : slots) * staged * t.geo[0].IW * 128.0;
        in_moved *= 1.0 + 1.05 * std::min(1.0, std::max(0.0, (under_way - 28e6) / 32e6));
        // and where pixels are no multiple of 64 bytes apart, half or three quarters of the chunks stand in two pieces of 64 (54 x 60 x 60, 384, 400 and
        // 392 -> 16: 46.7, 66.6 and 76.2 us in tiles of 7 columns, 35 MB, but 44.0, 48.5 and 50.5 in tiles of 4, 21 MB;
        // of 29 drawn passes that take tiles of 4 by it 21 are faster, up to 1.5 times, eight slower by up to 7 %)
        if (t.nch > 2 && (g.in_CH & 31)) in_moved *= 1.0 + (g.in_CH & 15 ? 0.6 : 0.4) * std::min(1.0, std::max(0.0, (under_way - 31e6) / 8e6));
    }
    const double move = (in_moved + (double)out_bytes) / 6.0e6;
    if (keep) {
        // Weights in LDS: tiles one after the other and the tensors' bytes, by whether there are more than 32 output channels and more than one
        // chunk (376 timings of 188 layers of up to 64 channels, 3 to 7 % rms; of two sets it is the
        // fastest in 30 and 42 % of the passes, by up to 26 %; those of one chunk set by which kernel is the faster)
        static const DmaTimes kKeep[2][2] = {{{0.857, 0, 0, 2.83, 0.426}, {1.330, 0, 0, 2.86, 0.419}}, {{0.64, 0, 0, 3.5, 0.9}, {2.72, 0, 0, 3.12, 0.447}}};
        const DmaTimes &c = kKeep[!narrow][t.nch - 1];
        *est = c.start + (t.rounds + (t.last > 0)) * c.chunk + c.bytes * move;
    } else {
        *est = (narrow ? kNarrow[first].start : cand.solo.start) + pow(pow(best, 1.5) + pow((narrow ? kNarrow[first].bytes : cand.solo.bytes) * move, 1.5), 1.0 / 1.5);
    }
    const int busy = t.last + t.pieces;
    *grid = t.rounds > 0 || busy > slots ? slots : busy;
    t.apart = t.m_fast ? m_tiles : 1;
    if (*grid % 8 == 0 && cand.at != 8 && (cand.mode != DM_S1 || !t.m_fast)) t.share = *grid / 8 > t.apart ? *grid / 8 / t.apart : 1;
    *out = t;
    return true;
}

typedef void (*DmaKernel)(const uint16_t *, uint16_t *, const uint16_t *, DmaArgs);

// The kernels of kDma by fused step. Only stride-1 passes are masked, and a backward pass has no ReLU of its own.
#define DM_ACTS(...) {&__VA_ARGS__, PC_ACT_NONE>, &__VA_ARGS__, PC_ACT_RELU>, &__VA_ARGS__, PC_ACT_RELU_MASK>}
#define DM_PAIR(BT, AT) {&pc_mfma_conv_dma_kernel<BT, PC_ACT_NONE, AT>, &pc_mfma_conv_dma_kernel<BT, PC_ACT_RELU, AT>, &pc_mfma_conv_dma_kernel<BT, PC_ACT_RELU_MASK, AT>}
static const DmaKernel kDmaKernels[kNumDma][3] = {
    DM_PAIR(8, 4), DM_PAIR(4, 4), DM_PAIR(7, 4),
    DM_ACTS(pc_mfma_conv_solo_kernel<DM_S1, 2, 4, 3), DM_ACTS(pc_mfma_conv_solo_kernel<DM_S1, 4, 4, 2), DM_ACTS(pc_mfma_conv_solo_kernel<DM_S1, 2, 2, 3),
    {&pc_mfma_conv_solo_kernel<DM_FWD2, 2, 4, 2, PC_ACT_NONE>, &pc_mfma_conv_solo_kernel<DM_FWD2, 2, 4, 2, PC_ACT_RELU>, nullptr},
    {&pc_mfma_conv_ring_kernel<PC_ACT_NONE>, &pc_mfma_conv_ring_kernel<PC_ACT_RELU>, nullptr},
    {&pc_mfma_conv_solo_kernel<DM_FWD2, 2, 2, 2, PC_ACT_NONE>, &pc_mfma_conv_solo_kernel<DM_FWD2, 2, 2, 2, PC_ACT_RELU>, nullptr},
    DM_ACTS(pc_mfma_conv_keep_kernel<4, 4, DM_KEEP_NBW),
    {&pc_mfma_conv_solo_kernel<DM_BWD2, 2, 4, 3, PC_ACT_NONE>, nullptr, nullptr},
    {&pc_mfma_conv_solo_kernel<DM_BWD2, 2, 2, 3, PC_ACT_NONE>, nullptr, nullptr}};
// For up to 32 output channels: the first three of kDma (by their place there), and code 50
static const DmaKernel kDmaNarrow[3][3] = {DM_PAIR(8, 2), DM_PAIR(4, 2), DM_PAIR(7, 2)};
static const DmaKernel kDmaKeepNarrow[3] = DM_ACTS(pc_mfma_conv_keep_kernel<2, 4, DM_KEEP_NBW);
#undef DM_ACTS
#undef DM_PAIR

static hipError_t launch_dma(DmaKernel kernel, pc_per_device_once &attr, int device, hipStream_t st, int grid, int threads, size_t lds, const uint16_t *in,
                             uint16_t *out, const uint16_t *wz, const DmaArgs &g)
{
    if (pc_once_pending(attr, device)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, DM_LDS_MAX);
        if (e != hipSuccess) return e;
        pc_once_done(attr, device);
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3((unsigned)threads), lds, st, in, out, wz, g);
    return hipGetLastError();
}

// pcfg: -1 or a code of kDma; lgCG: -1 or the wavefronts side by side (log2), on return those of the plan taken. *launched stays 0
// where no kernel takes the launch or no estimate is below limit (us); it becomes the kernel's code.
pc_status pc_run_mfma_conv_dma(pc_ctx *ctx, int pcfg, int *lgCG, double limit, const MfmaArgs &g0, bool flip, const uint16_t *in, uint16_t *out,
                               const uint16_t *wz, int *launched, int act)
{
    *launched = 0;
    if ((g0.in_CH & 7) || (g0.out_CH & 7) || !pc_direct_loads(in)) return PC_OK;
    const int mode = g0.oscale == 2 ? DM_BWD2 : g0.lstep == 2 ? DM_FWD2 : DM_S1;
    DmaArgs best;
    size_t best_lds = 0;
    int best_grid = 0, best_k = -1;
    double best_est = limit;
    for (int k = 0; k < kNumDma; ++k) {
        if (kDma[k].mode != mode || !kDmaKernels[k][act] || (pcfg >= 0 && pcfg != kDma[k].code)) continue;
        for (int lg = *lgCG < 0 ? 0 : *lgCG; lg <= (*lgCG < 0 ? 2 : *lgCG); ++lg) {
            DmaArgs t;
            size_t lds;
            int grid;
            double est;
            if (!plan_dma(g0, flip, kDma[k], lg, &t, &lds, &grid, &est, ctx->num_cu)) continue;
            if (est < best_est) { best = t; best_lds = lds; best_grid = grid; best_k = k; best_est = est; }
        }
    }
    if (best_k < 0) return PC_OK;
    const DmaCand &c = kDma[best_k];
    static pc_per_device_once attr[kNumDma][3], attr_narrow[4][3];
    const bool narrow = (c.nbuf == 1 || c.nbuf == 4) && g0.out_CH <= 32;
    const int row = c.nbuf == 4 ? 3 : best_k;
    const hipError_t e = launch_dma(!narrow ? kDmaKernels[best_k][act] : c.nbuf == 4 ? kDmaKeepNarrow[act] : kDmaNarrow[best_k][act], narrow ? attr_narrow[row][act] : attr[best_k][act], ctx->device, ctx->stream, best_grid, c.nbuf == 1 ? 256 : 512, best_lds, in, out,
                                    wz, best);
    *launched = c.code;
    *lgCG = best.lgCG;
    if (c.at == 8) pc_note_kernel(ctx, "pc_mfma_conv_ring_kernel<%d>", act);
    else if (c.nbuf == 1) pc_note_kernel(ctx, "pc_mfma_conv_dma_kernel<%d, %d, %d>", c.bt, act, narrow ? 2 : 4);
    else if (c.nbuf == 4) pc_note_kernel(ctx, "pc_mfma_conv_keep_kernel<%d, %d, %d, %d>", narrow ? 2 : 4, c.bt, DM_KEEP_NBW, act);
    else pc_note_kernel(ctx, "pc_mfma_conv_solo_kernel<%d, %d, %d, %d, %d>", c.mode, c.at, c.bt, c.nbuf, act);
    return pc_hip_check(ctx, e, "MFMA conv (direct loads) launch");
}
