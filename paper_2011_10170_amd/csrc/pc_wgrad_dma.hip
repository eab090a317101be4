// Backward-weight on the matrix cores (bf16 layers), operands straight from NHWC rows in LDS (see pc_wgrad_mfma.hip for the pass
// itself, the splits of the pixels and the partial planes).
#include "pc_wgrad_dma.h"

#include <math.h>

// dW[t][f][c] = sum over output pixels of dy[pixel][f] * x[pixel shifted by tap t][c]. A workgroup of 4 wavefronts owns a tile of 64
// filters x 64 channels, a wavefront 32 x 32 of it for all nine taps (144 accumulator registers), and walks tiles of TR rows x TC
// columns of output pixels; two workgroups share a CU, one loads (or writes its sums) while the other multiplies.
//   Instruction: v_mfma_f32_16x16x32_bf16, whose rate on dense operands (1.98 PFLOP/s fed from LDS; power) is above that of the 32x32x16
//     form (1.71). Its 32 reduction entries are 32 rows of one column.
//   gfx950's transposing LDS read (ds_read_b64_tr_b16: 16 lanes read 4 rows of 16 values and get 4 values of one column each) makes
//     the operand, 8 pixels of one channel per lane, from pixel rows as they lie in memory: nothing is transposed in registers, and
//     the tiles are brought to LDS by direct loads.
//   The x operands of a column (3 tap rows x 2 halves of the channels) are multiplied with dy of the output columns they are tap columns
//     0, 1 and 2 of, while the next column's are read: a step of 36 matrix instructions reads 6 x operands and 2 of dy.
//   Rows: the output rows of all images in order; the x rows of images of H + 1 rows, one zero row between two of them, so a tile
//     covers any TR rows. Rows past the last one are zeros on both sides.
//   A staged row is its pixels' 128 bytes (64 channels) and a pad, so that the rows a transposing read takes start in different banks.
//   Layers whose last tile of 64 filters or channels would be half empty take tiles of 32: the wavefronts that are then left over share the
//     tile's pixels (rows or columns of it), and their sums are added in LDS. 34 images 209 x 208, 32 -> 8: 65 -> 38 us; 50 images
//     80 x 80, 144 -> 80: 98 -> 80.
//   What a small layer's call spends (5 images 14 x 14, 48 -> 24, 8.5 us; stamps of one lane): arguments and zeros 0.65, first loads 1.9,
//     products 0.9 to 2.6 (a tile of 64 rows is 16 steps, of 32 x 1 one), look-up table 0.8, pick of the kept taps and stores 2.3. Hence
//     small tiles and many splits for small layers, the table's lines touched at the start, a pick of 41 instructions a kernel instead
//     of 54, and arguments of 272 bytes: 13 images 33 x 47, 40 -> 72 13.6 -> 12.4 us with the partial planes added.
#define WD_OOB 0x80000000u

typedef short i16x4 __attribute__((ext_vector_type(4)));

// Lanes of mask x 16 bytes from a buffer to LDS at lds_off + 16 * lane; an offset past the buffer's end writes zeros. Only where all
// lanes are active: exec is as it was afterwards. (m0: see dm_load.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void wd_load(const v4u32 &rsrc, uint32_t voff, int soff, int lds_off, uint64_t mask)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds\n\ts_mov_b64 exec, -1"
                 :: "s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff), "s"(mask) : "memory", "m0");
}
#pragma clang diagnostic pop

// A launch argument that stays in its register: the compiler would read it again from memory wherever it is used.
__device__ __forceinline__ int wd_keep(int v)
{
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ v4u32 wd_rsrc(const void *p, uint32_t bytes)
{
    const uint64_t a = (uint64_t)p;
    const v4u32 r = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu)),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
    return r;
}

// 8 reduction entries of one row / column of a matrix operand: two transposing reads of 4 pixel rows each
__device__ __forceinline__ bf16x8 wd_frag(const unsigned char *p0, const unsigned char *p1)
{
    typedef __attribute__((address_space(3))) i16x4 *lds4;
    const i16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p0)), b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p1));
    const short __attribute__((ext_vector_type(8))) v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    bf16x8 o;
    __builtin_memcpy(&o, &v, 16);
    return o;
}

// (a uniform choice between registers, which cannot be indexed)
__device__ __forceinline__ f32x4 wd_pick(bool second, const f32x4 &p, const f32x4 &q)
{
    f32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = second ? q[i] : p[i];
    return o;
}

// lin: index of the workgroup in the layer's grid of gx x gy tiles x ksplit splits (x fastest).
// FW, CW: wavefronts side by side along the filters and the channels of the workgroup's tile; the other 4 / (FW * CW) share the tile's pixels.
template <int ST, int FW, int CW>
__device__ __forceinline__ void pc_wgrad_dma_body(const uint16_t *__restrict__ x, const uint16_t *__restrict__ dy, const WgradDmaArgs &a,
                                                  const uint32_t *__restrict__ kinfo, float *__restrict__ partial, float *__restrict__ dw, int lin, int gx)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int PW = 4 / (FW * CW), XB = 64 * CW, DB = 64 * FW;      // bytes per staged pixel of x and of dy
    constexpr int XL = 4 * CW, DL = 4 * FW;                             // lanes of a direct load per pixel
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups of an XCD share as few pixel splits as possible (as in pc_mfma_wgrad_ws_body)
    int bz = lin >> 3, tile = lin & 7;
    if (a.place == WD_PLACE_MANY) {              // 8, 16, .. splits: an XCD's in order
        const int q = (int)pc_udiv((uint32_t)bz, a.mg_T);
        const int xcd = tile;
        tile = bz - q * a.T;
        bz = q * 8 + xcd;
    } else if (a.place == WD_PLACE_FEW) {        // 1, 2 or 4 splits: 8 / ksplit XCDs share one
        const int xcd = tile;
        tile = ((bz << 3) >> a.lgks) + (xcd >> a.lgks);
        bz = xcd & (a.ksplit - 1);
    } else {
        bz = (int)pc_udiv((uint32_t)lin, a.mg_T);
        tile = lin - bz * a.T;
    }
    const int by = (int)pc_udiv((uint32_t)tile, a.mg_gx), bx = tile - by * gx;
    const int c0 = bx * (32 * CW), f0 = by * (32 * FW);
    const int fw = w % FW, cw = w / FW % CW, pw = w / (FW * CW);
    const v4u32 xs = wd_rsrc(x, a.x_bytes), ds = wd_rsrc(dy, a.dy_bytes);
    const int x_row = wd_keep(a.W * a.C * 2), d_row = wd_keep(a.Wo * a.F * 2);       // bytes per row
    const int H1 = wd_keep(a.H + 1), nimg = wd_keep(a.N), rows = wd_keep(a.rows), nrow = wd_keep(a.nrow), TR = wd_keep(a.TR), TC = a.TC, IW = a.IW,
              RPx = wd_keep(a.RPx), RPd = wd_keep(a.RPd), dy_off = a.dy_off, n_ktiles = a.n_ktiles, ksplit = a.ksplit;
    // The wavefronts that share pixels: 1 << lgPC side by side, each with NC columns, the others below each other
    const int col0 = PW > 1 ? (pw & ((1 << a.lgPC) - 1)) * a.NC : 0, left = TC - col0, nc = PW > 1 ? wd_keep(left < a.NC ? left : a.NC) : TC,
              ncx = PW > 1 ? wd_keep(nc + 2) : IW;      // (two numbers to the compiler)
    // lanes of the loads of a row
    const uint64_t mask_a = IW * XL >= 64 ? ~0ull : (1ull << (XL * IW)) - 1, mask_b = IW * XL > 64 ? ~0ull >> (128 - XL * IW) : 0,
                   mask_d = TC * DL >= 64 ? ~0ull : (1ull << (DL * TC)) - 1;
    const bool x_ok = c0 + (lane & (XL - 1)) * 8 < a.C, d_ok = f0 + (lane & (DL - 1)) * 8 < a.F;
    // where this lane's transposing reads start inside 4 pixels' rows (4 of 16 channels or filters), and the first row it reads
    // (stride 2: the 32 reduction entries are 16 rows of two columns that follow each other, for less LDS per tile)
    constexpr int KROWS = ST == 1 ? 32 : 16;
    const int sub = (lane & 3) * 8, krow = 8 * ((lane >> 4) & (KROWS / 8 - 1)) + ((lane & 15) >> 2), kcol = ST == 1 ? 0 : lane >> 5;
    const int h_first = PW > 1 ? (left > 0 ? (pw >> a.lgPC) * KROWS : TR) : 0, h_step = PW > 1 ? wd_keep((PW >> a.lgPC) * KROWS) : KROWS;

    // The look-up table of the epilogue comes from L2 then: every 128-byte line of the tile's rows is touched now.
    uint32_t touched = 0;
    if ((int)threadIdx.x < 32 * FW * CW) {
        const int f = f0 + (int)threadIdx.x / CW, c = c0 + (int)threadIdx.x % CW * 32;
        if (f < a.F && c < a.C) touched = kinfo[(int64_t)f * a.C + c];
    }

    f32x4 acc[9][2][2];       // tap, filter half, channel half of the wavefront's 32 x 32
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int kt = bz; kt < n_ktiles; kt += ksplit) {
        const int tr = (int)pc_udiv((uint32_t)kt, a.mg_tc), x0 = (kt - tr * a.tiles_c) * TC, r0 = tr * TR;
        const int n0 = (int)pc_udiv((uint32_t)r0, a.mg_Ho), V0 = n0 * H1 + (r0 - n0 * a.Ho) * ST;
        if (kt != bz) asm volatile("s_barrier" ::: "memory");      // every wavefront has read what the loads replace
        __builtin_amdgcn_s_setprio(3);
        {
            // a wavefront's load brings 64 / XL pixels of a row, the x columns past them come in a second one
            uint32_t vx[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int xx = x0 * ST - 1 + p * (64 / XL) + lane / XL;
                vx[p] = x_ok && (unsigned)xx < (unsigned)a.W ? (uint32_t)(xx * a.C + c0 + (lane & (XL - 1)) * 8) * 2u : WD_OOB;
            }
            const uint32_t vd = d_ok && x0 + lane / DL < a.Wo ? (uint32_t)((x0 + lane / DL) * a.F + f0 + (lane & (DL - 1)) * 8) * 2u : WD_OOB;
            // row y of an image is row y + 1 of the padded image, row 0 is zeros
            int v = V0 + w, n = (int)pc_udiv((uint32_t)v, a.mg_H1), y1 = v - n * H1, at = w * RPx;
            for (int row = w; row < nrow; row += 4) {
                const bool ok = y1 > 0 && n < nimg;
                const int so = ok ? (v - n - 1) * x_row : 0;
                wd_load(xs, ok ? vx[0] : WD_OOB, so, at, mask_a);
                if (mask_b) wd_load(xs, ok ? vx[1] : WD_OOB, so, at + 1024, mask_b);
                at += 4 * RPx;
                v += 4;
                for (y1 += 4; y1 >= H1; y1 -= H1) ++n;
            }
            at = dy_off + w * RPd;
            int so = (r0 + w) * d_row;
            for (int row = w; row < TR; row += 4) {
                const bool ok = r0 + row < rows;
                wd_load(ds, ok ? vd : WD_OOB, ok ? so : 0, at, mask_d);
                at += 4 * RPd;
                so += 4 * d_row;
            }
        }
        __builtin_amdgcn_s_setprio(0);
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        for (int hh = h_first; hh < TR; hh += h_step) {
            const unsigned char *pr[3][2], *pd[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int k = hh + krow + 4 * q, rho = r0 + k, n = (int)pc_udiv((uint32_t)rho, a.mg_Ho);
                pr[0][q] = lds + (n * H1 + (rho - n * a.Ho) * ST - V0) * RPx + cw * 64 + sub + (kcol + col0) * (ST * XB);
                pr[1][q] = pr[0][q] + RPx;
                pr[2][q] = pr[1][q] + RPx;
                pd[q] = lds + dy_off + k * RPd + fw * 64 + sub + (kcol + col0) * DB;
            }
            bf16x8 xq[3][2], dq[4][2];
            auto read_x = [&](int r, int h, int col) __attribute__((always_inline)) { xq[r][h] = wd_frag(pr[r][0] + col * XB + h * 32, pr[r][1] + col * XB + h * 32); };
            auto read_d = [&](int col) __attribute__((always_inline)) {
#pragma unroll
                for (int h = 0; h < 2; ++h) dq[col & 3][h] = wd_frag(pd[0] + col * DB + h * 32, pd[1] + col * DB + h * 32);
            };
            read_d(0);
#pragma unroll
            for (int i = 0; i < 6; ++i) read_x(i >> 1, i & 1, 0);
            if constexpr (ST == 2) {
                // pairs of output columns: tap column q of the pair from column c is the pair of x columns 2c + q and 2c + q + 2
#pragma unroll
                for (int u = 0; u < 9; ++u) {
                    const int c = 2 * (u / 3), q = u % 3;
                    if (c < nc) {
                        if (q == 0 && u + 3 < 9) read_d(c + 2);
                        if (u == 3) __builtin_amdgcn_s_setprio(1);
                        if (u == 6) __builtin_amdgcn_s_setprio(2);
                        const int next = q < 2 ? 2 * c + q + 1 : 2 * c + 4;
#pragma unroll
                        for (int i = 0; i < 6; ++i) {
#pragma unroll
                            for (int h = 0; h < 2; ++h)
                                acc[(i >> 1) * 3 + q][h][i & 1] =
                                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(dq[c & 3][h], xq[i >> 1][i & 1], acc[(i >> 1) * 3 + q][h][i & 1], 0, 0, 0);
                            if (u + 1 < 9) read_x(i >> 1, i & 1, next);
                        }
#pragma unroll
                        for (int i = 0; i < 6; ++i) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                            if (u + 1 < 9) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                continue;
            }
            constexpr int LAST = 9;              // last x column of 8 output columns
            // (the columns left and right of the map are zeros: nothing to add. 7 x 7 maps: 19 of 21 products per row)
            const bool left = x0 + col0 > 0;
            const int xend = wd_keep(x0 + col0 + nc < a.Wo ? ncx : ncx - 1 - (x0 + col0 + nc - a.Wo));
#pragma unroll
            for (int X = 0; X <= LAST; ++X) {
                if (X < xend) {
                    // (past the tile's last column, up to three columns on: the row's pad, the next row or the room the plan leaves after
                    // the last one; not used. The x columns past a row's last one run into the next row, or into dy.)
                    if (X + 1 < 8) read_d(X + 1);
                    if (X == 3) __builtin_amdgcn_s_setprio(1);
                    if (X == 6) __builtin_amdgcn_s_setprio(2);
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const int j = X - q;                              // output column X is tap column q of
                        if (j < 0 || j > 7) continue;
                        const bool final = j == 0 || q == 2;              // the last taps column X takes part in: its operands are replaced
                        if (X == 0 && !left) {
#pragma unroll
                            for (int i = 0; i < 6; ++i) read_x(i >> 1, i & 1, 1);
                        } else if (j < nc) {
#pragma unroll
                            for (int i = 0; i < 6; ++i) {
#pragma unroll
                                for (int h = 0; h < 2; ++h)
                                    acc[(i >> 1) * 3 + q][h][i & 1] =
                                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(dq[j & 3][h], xq[i >> 1][i & 1], acc[(i >> 1) * 3 + q][h][i & 1], 0, 0, 0);
                                if (final && X < LAST) read_x(i >> 1, i & 1, X + 1);
                            }
#pragma unroll
                            for (int i = 0; i < 6; ++i) {
                                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                                if (final && X < LAST) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            }
        }
    }
    __builtin_amdgcn_s_setprio(3);
    asm volatile("" :: "v"(touched));
    // Wavefronts that shared pixels add their sums through LDS, halves of the 32 x 32 at a time: partners swap the filter halves (a wavefront
    // keeps one), of four then also the channel halves. What is left to write is 4 / PW blocks of 16 x 16, block b in acc[..][b >> 1][b & 1].
    int fh = 0, ch = 0;       // the halves kept
    if constexpr (PW > 1) {
        f32x4 *mine = reinterpret_cast<f32x4 *>(lds) + w * (18 * 64) + lane;
        const f32x4 *theirs = reinterpret_cast<const f32x4 *>(lds) + (w ^ (FW * CW)) * (18 * 64) + lane;
        fh = pw & 1;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                mine[(t * 2 + c) * 64] = wd_pick(fh == 0, acc[t][0][c], acc[t][1][c]);
                acc[t][0][c] = wd_pick(fh != 0, acc[t][0][c], acc[t][1][c]);
                __builtin_amdgcn_sched_barrier(0);
            }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                acc[t][0][c] += theirs[(t * 2 + c) * 64];
                if (t % 3 == 2) __builtin_amdgcn_sched_barrier(0);
            }
    }
    if constexpr (PW > 2) {
        f32x4 *mine = reinterpret_cast<f32x4 *>(lds) + w * (9 * 64) + lane;
        const f32x4 *theirs = reinterpret_cast<const f32x4 *>(lds) + (w ^ 2) * (9 * 64) + lane;
        ch = pw >> 1;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            mine[t * 64] = wd_pick(ch == 0, acc[t][0][0], acc[t][0][1]);
            acc[t][0][0] = wd_pick(ch != 0, acc[t][0][0], acc[t][0][1]);
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t][0][0] += theirs[t * 64];
    }
    // Epilogue: a lane holds all nine taps of its 16 / PW kernels; the 4 kept ones of a kept kernel move down in place and are written in
    // compact slot order. (Tap by tap from the last: a kept one becomes the first of the kept values and moves the others up.)
    constexpr int NK = 16 / PW;
    float *pout = a.ksplit > 1 ? partial + (int64_t)bz * a.pstride * 4 : dw;
    uint32_t info[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) {       // (all loads at once: clamped, not under a condition)
        const int f = f0 + fw * 32 + (PW > 1 ? fh : k >> 3) * 16 + 4 * (lane >> 4) + (k & 3), c = c0 + cw * 32 + (PW > 2 ? ch : (k >> 2) & 1) * 16 + (lane & 15);
        const bool in = f < a.F && c < a.C;
        const uint32_t u = kinfo[in ? (uint32_t)f * (uint32_t)a.C + (uint32_t)c : 0u];
        info[k] = in ? u : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        uint32_t m = info[k] << 23;
#pragma unroll
        for (int t = 8; t >= 0; --t) {
            const bool kept = __builtin_uadd_overflow(m, m, &m);       // (tap t's bit: one addition that shifts it out)
            o.w = kept ? o.z : o.w;
            o.z = kept ? o.y : o.z;
            o.y = kept ? o.x : o.y;
            o.x = kept ? acc[t][k >> 3][(k >> 2) & 1][k & 3] : o.x;
        }
        if (info[k] != 0xFFFFFFFFu) *reinterpret_cast<float4 *>(pout + (int64_t)(info[k] >> 9) * 4) = o;
    }
}

template <int ST>
__device__ __forceinline__ void pc_wgrad_dma_layer(const WgradDmaLayer &y, int lin)
{
    switch (y.a.waves) {
    case 0: pc_wgrad_dma_body<ST, 2, 2>(y.x, y.dy, y.a, y.kinfo, y.partial, y.dw, lin, y.gx); break;
    case 1: pc_wgrad_dma_body<ST, 1, 2>(y.x, y.dy, y.a, y.kinfo, y.partial, y.dw, lin, y.gx); break;
    case 2: pc_wgrad_dma_body<ST, 2, 1>(y.x, y.dy, y.a, y.kinfo, y.partial, y.dw, lin, y.gx); break;
    default: pc_wgrad_dma_body<ST, 1, 1>(y.x, y.dy, y.a, y.kinfo, y.partial, y.dw, lin, y.gx); break;
    }
}

// One layer. Its arguments are 272 bytes; those of a network (below) are 4 KiB, which a launch copies and every workgroup searches.
template <int ST, int FW, int CW>
__global__ void __launch_bounds__(256, 2) pc_mfma_wgrad_dma_kernel(WgradDmaOne g)
{
    const WgradDmaLayer &y = g.layer[0];
    pc_wgrad_dma_body<ST, FW, CW>(y.x, y.dy, y.a, y.kinfo, y.partial, y.dw, (int)blockIdx.x, y.gx);
}

// Wavefronts along the filters and the channels of a workgroup's tile
static const struct { int fw, cw, lgPW; } kWaves[WD_WAVES] = {{2, 2, 0}, {1, 2, 1}, {2, 1, 1}, {1, 1, 2}};     // (lgPW: log2 of those that share pixels)

static int wd_placed(int T, int ks) { return ks % 8 == 0 ? WD_PLACE_MANY : 8 % ks == 0 && T % (8 / ks) == 0 ? WD_PLACE_FEW : WD_PLACE_PLAIN; }

// The part of a layer's plan that does not depend on its tiles; false when the layer is outside what the kernel takes.
static bool wd_layer(const pc_conv_desc *d, int64_t nslots, WgradDmaArgs &a)
{
    memset(&a, 0, sizeof(a));
    const int st = d->stride;
    a.N = d->N; a.H = d->H; a.W = d->W; a.C = d->C; a.F = d->F; a.stride = st;
    a.Ho = (d->H - 1) / st + 1; a.Wo = (d->W - 1) / st + 1;
    const int64_t xb = (int64_t)a.N * a.H * a.W * a.C * 2, db = (int64_t)a.N * a.Ho * a.Wo * a.F * 2, rows = (int64_t)a.N * a.Ho;
    if ((d->C & 7) || (d->F & 7) || xb >= ((int64_t)1 << 31) || db >= ((int64_t)1 << 31) || rows >= (1 << 24)) return false;
    // (pc_udiv is exact below 2^32 / divisor. A tile of 128 rows ends up to 127 rows past the last image: beyond the 64 here only where Ho is above
    // 255, as the rows are below 2^24, and those rows leave remainders below 127, which the quotient is exact for, too.)
    if ((rows + 64) * a.Ho >= ((int64_t)1 << 32) || ((int64_t)a.N + 66) * (a.H + 1) * (a.H + 1) >= ((int64_t)1 << 32)) return false;
    a.x_bytes = (uint32_t)xb; a.dy_bytes = (uint32_t)db;
    a.rows = (int)rows;
    a.pstride = (int32_t)nslots;
    a.mg_Ho = pc_udiv_magic(a.Ho); a.mg_H1 = pc_udiv_magic(a.H + 1);
    return true;
}

// The plan with this arrangement of the wavefronts, 1 << lgPC of those that share pixels side by side with nc columns each, in tiles of TR
// rows; false when it does not fit.
static bool wd_tile(const WgradDmaArgs &layer, int waves, int lgPC, int TR, int nc, WgradDmaPlan *out)
{
    WgradDmaPlan p;
    p.a = layer;
    WgradDmaArgs &a = p.a;
    const int st = a.stride, krows = st == 1 ? 32 : 16, fw = kWaves[waves].fw, cw = kWaves[waves].cw, lgPW = kWaves[waves].lgPW, XB = 64 * cw, DB = 64 * fw;
    a.waves = waves; a.lgPC = lgPC; a.TR = TR; a.NC = nc;
    // (columns of wavefronts past the map's last one are not staged)
    const int wide = (a.Wo + st - 1) / st * st;
    a.TC = nc << lgPC < wide ? nc << lgPC : wide;
    a.IW = st * (a.TC - 1) + 3;
    if (a.TC * DB > 1024 || a.IW * XB > 2048) return false;       // a row of dy is one direct load, a row of x at most two
    // image boundaries inside a tile (tiles start at multiples of TR); rows past the last image lie as if more images followed
    const int cross = a.Ho % TR == 0 ? 0 : TR % a.Ho == 0 ? TR / a.Ho - 1 : (TR - 1 + a.Ho - 1) / a.Ho;
    a.nrow = st * (TR - 1) + 3 + cross * (a.H + 1 - st * a.Ho);
    a.RPx = a.IW * XB + (st == 1 ? 32 : 16);
    a.dy_off = a.nrow * a.RPx;
    // columns of dy that are read past the end of a row: three, none past a wavefront's eighth (stride 1), or the next pair (stride 2)
    const int past = st == 1 ? (nc + 3 < 8 ? 3 : 8 - nc) : nc < 6 ? 2 : 0;
    for (int pad = 32;; pad = 0) {
        a.RPd = a.TC * DB + pad;
        p.lds = (size_t)(a.dy_off + TR * a.RPd + (past * DB > pad ? past * DB - pad : 0));
        if (p.lds <= WD_LDS_MAX) break;
        if (pad == 0) return false;
    }
    if (lgPW && p.lds < WD_LDS_SUMS) p.lds = WD_LDS_SUMS;
    a.tiles_c = (a.Wo + a.TC - 1) / a.TC;
    a.n_ktiles = (a.rows + TR - 1) / TR * a.tiles_c;
    if ((int64_t)a.n_ktiles * a.tiles_c >= ((int64_t)1 << 32)) return false;
    a.mg_tc = pc_udiv_magic(a.tiles_c);
    p.ct = (a.C + 32 * cw - 1) / (32 * cw);
    p.ft = (a.F + 32 * fw - 1) / (32 * fw);
    p.steps = (TR / krows >> (lgPW - lgPC)) * (nc / st);
    p.loads = (a.nrow * (a.IW * XB > 1024 ? 2 : 1) + TR + 3) / 4;
    const double load = 0.0893 * p.loads, mul = 0.498 * p.steps;
    p.tile_us = 0.574 + sqrt(load * load + mul * mul);
    p.end_us = 2.2 * (0.28 * (4 >> lgPW) + (lgPW == 0 ? 0.0 : lgPW == 1 ? 1.25 : 1.87));
    a.ksplit = 0;
    *out = p;
    return true;
}

// `use` is called with every plan that fits (of one arrangement of the wavefronts: only >= 0). Tiles of 32 filters or channels are for layers
// whose last tile of 64 would be half empty: elsewhere they were the fastest by 0.6 % on average.
template <class Use> static void wd_plans(const WgradDmaArgs &layer, int only, Use use)
{
    const int st = layer.stride, krows = st == 1 ? 32 : 16;
    WgradDmaPlan p;
    for (int w = 0; w < WD_WAVES; ++w) {
        if (only >= 0 ? w != only : (kWaves[w].cw == 1 && (-layer.C & 63) < 32) || (kWaves[w].fw == 1 && (-layer.F & 63) < 32)) continue;
        const int lgPW = kWaves[w].lgPW;
        for (int lgPC = 0; lgPC <= lgPW; ++lgPC)
            for (int TR = krows << (lgPW - lgPC); TR <= (lgPW ? 128 : 64); TR += krows << (lgPW - lgPC))
                for (int nc = st; nc <= (st == 1 ? 8 : 6) && (nc - st) << lgPC < layer.Wo; nc += st)
                    if (wd_tile(layer, w, lgPC, TR, nc, &p)) use(p);
    }
}

static int32_t wd_code(const WgradDmaPlan &p) { return p.a.waves | p.a.lgPC << 2 | p.a.TR / 16 << 4 | p.a.NC << 8 | p.a.ksplit << 12; }
static bool wd_decode(const WgradDmaArgs &layer, int32_t c, WgradDmaPlan *out)
{
    if (!wd_tile(layer, c & 3, (c >> 2) & 3, ((c >> 4) & 15) * 16, (c >> 8) & 15, out)) return false;
    out->a.ksplit = c >> 12;
    return true;
}

bool pc_wgrad_dma_plan(const pc_conv_desc *d, int64_t nslots, int32_t *choice, WgradDmaPlan *out)
{
    WgradDmaArgs layer;
    if (!wd_layer(d, nslots, layer)) return false;
    if (*choice >= 0) return wd_decode(layer, *choice, out);
    double best = 1e30;
    wd_plans(layer, -1, [&](const WgradDmaPlan &p) {
        const double t = (double)p.ct * p.ft * p.a.n_ktiles * p.tile_us;
        if (t < best) { best = t; *out = p; }
    });
    if (best < 1e30) *choice = wd_code(*out);
    return best < 1e30;
}

bool pc_wgrad_dma_plan_one(const pc_conv_desc *d, int64_t nslots, double kept, int num_cu, int waves, int32_t *choice, WgradDmaPlan *out)
{
    WgradDmaArgs layer;
    if (!wd_layer(d, nslots, layer)) return false;
    if (choice && *choice >= 0) return wd_decode(layer, *choice, out);
    // Estimated time (us): a start, the pixel tiles of a workgroup one after the other (a lone one on its CU: a wait, loads and products in
    // sequence; two sharing it: loads and products overlap), the sums of wavefronts that share pixels and the pick of the kept taps of
    // 16 x 16 blocks, the tensors' bytes; the partial planes and their launch. Of splits that leave the workgroups of an XCD without shared
    // pixels (WD_PLACE_PLAIN) every staged byte comes from beyond its L2: 144 -> 80, 50 images of 80 x 80, 34 splits of tiles of 32 x 32 186 us,
    // 32 splits 95. Fitted to 25000 timings of 160 layers (7 % rms), on which the choice is 3.5 % behind the fastest, the worst 17 % (on the
    // 67 of profiles/wgrad_plan_timings_bf16.csv 3.7 and 19 %);
    // one tile of 64 x 64, the pixel tile of the best throughput and as many splits as fill the chip were 12 % behind.
    const double bytes = (double)layer.x_bytes + layer.dy_bytes;
    double best = 1e30;
    wd_plans(layer, waves, [&](const WgradDmaPlan &p) {
        const int T = p.ct * p.ft;
        const double lone = 0.526 + 0.068 * p.loads + 0.319 * p.steps;
        const double staged = ((double)p.a.nrow * p.a.IW * kWaves[p.a.waves].cw + (double)p.a.TR * p.a.TC * kWaves[p.a.waves].fw) * 64.0;
        int last = 0;
        for (int places = 2 * num_cu; places >= num_cu / 4; places >>= 1)
            for (int even = 0; even < 2; ++even) {
                int ks = places / T < p.a.n_ktiles ? places / T : p.a.n_ktiles;
                if (ks < 1) ks = 1;
                if (even) ks = ks >= 8 ? ks & ~7 : ks >= 4 ? 4 : ks >= 2 ? 2 : 1;
                if (ks == last) continue;
                last = ks;
                const int u = (p.a.n_ktiles + ks - 1) / ks, rounds = (T * ks + 2 * num_cu - 1) / (2 * num_cu);
                const double t = 3.25 + (T * ks <= num_cu ? u * lone + p.end_us / 2.2 : rounds * (u * p.tile_us + p.end_us));
                const double moved = 0.168e-6 * bytes + (wd_placed(T, ks) == WD_PLACE_PLAIN ? 0.112e-6 * staged * T * ks * u : 0.0);
                const double us = cbrt(t * t * t + moved * moved * moved) + (ks > 1 ? 2.5 + 10.7e-6 * ks * kept : 0.0);
                if (us < best) { best = us; *out = p; out->a.ksplit = ks; out->us = us; }
            }
    });
    if (best < 1e30 && choice) *choice = wd_code(*out);
    return best < 1e30;
}

// Where the workgroups of a layer find their tile and split.
static void wd_place(WgradDmaLayer &y)
{
    WgradDmaArgs &a = y.a;
    a.T = y.gx * y.gy;
    a.mg_T = pc_udiv_magic(a.T);
    a.mg_gx = pc_udiv_magic(y.gx);
    a.lgks = a.ksplit >= 4 ? 2 : a.ksplit == 2;
    a.place = wd_placed(a.T, a.ksplit);
}

template <class Args>
static pc_status wd_launch(pc_ctx *ctx, void (*kernel)(Args), pc_per_device_once &attr, const Args &g, size_t lds, int more = 0)
{
    if (pc_once_pending(attr, ctx->device)) {
        PC_HIP(ctx, hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, WD_LDS_MAX));
        pc_once_done(attr, ctx->device);
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(g.blk0[g.n] + more)), dim3(256), lds, ctx->stream, g);
    return pc_hip_check(ctx, hipGetLastError(), "MFMA bwd_weight (direct loads) launch");
}

pc_status pc_wgrad_dma_launch(pc_ctx *ctx, WgradDmaOne &g, size_t lds)
{
    wd_place(g.layer[0]);
    typedef void (*One)(WgradDmaOne);
#define WD_ONES(st) {&pc_mfma_wgrad_dma_kernel<st, 2, 2>, &pc_mfma_wgrad_dma_kernel<st, 1, 2>, &pc_mfma_wgrad_dma_kernel<st, 2, 1>, &pc_mfma_wgrad_dma_kernel<st, 1, 1>}
    static const One kernels[2][WD_WAVES] = {WD_ONES(1), WD_ONES(2)};
#undef WD_ONES
    static pc_per_device_once attr[2][WD_WAVES];
    const WgradDmaArgs &a = g.layer[0].a;
    pc_note_kernel(ctx, "pc_mfma_wgrad_dma_kernel<%d, %d, %d>", a.stride, kWaves[a.waves].fw, kWaves[a.waves].cw);
    return wd_launch(ctx, kernels[a.stride - 1][a.waves], attr[a.stride - 1][a.waves], g, lds);
}

// ------------------------------------------------------------------ few input channels
// Backward-weight of a layer with at most 4 input channels (the first of a network). The taps and channels of one tap row are the 16 columns of one
// matrix operand: the input is staged as pixels of 4 channels (8 bytes), so the 4 x 4 values of 4 pixels side by side are 32 consecutive
// bytes, and a transposing read of 4 such rows makes column 4 * s + c of the operand (s = 3 is computed and dropped). 32 rows of one column of
// output pixels are a step: 3 tap rows x F / 16 instructions. What bounds it is one pass over dy: 32 images 224 x 224, 3 -> 64 (205 MB)
// 40 us (5.4 TB/s) for 79 of the general kernel and 11 of the 8-channel copy of x that it reads.
//   A workgroup walks tiles of 32 rows x TC columns; dy comes to one LDS buffer by direct loads and x (3 values of 64 of dy's) through
//   registers while the tile in the other buffer is multiplied. Wavefront w takes columns w, w + 4, ..; sums are added through LDS at the end.
//   Tiles are small (16 KiB of dy): with 32 KiB 11 us more, and a pixel of x is one load of 8 bytes: with one per channel 2 us more.
#define TW_ROWS 32

// NF: blocks of 16 filters, XP: pixels of x per thread and tile at most
template <int NF, int XP>
__device__ __forceinline__ void pc_thin_wgrad_body(const uint16_t *__restrict__ x, const uint16_t *__restrict__ dy, const ThinWgradArgs &a,
                                                   const uint32_t *__restrict__ kinfo, float *__restrict__ out, int wg, int G, int f0, unsigned char *lds)
{
    constexpr int DB = NF > 2 ? 128 : 64, DL = DB / 16;      // bytes and lanes of a direct load per pixel of dy
    const int lane = threadIdx.x & 63, tid = (int)threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const v4u32 ds = wd_rsrc(dy, a.dy_bytes);
    const int d_row = a.Wo * a.F * 2, H1 = a.H + 1;
    const uint64_t mask_c = a.C == 4 ? ~0ull : (1ull << (16 * a.C)) - 1;
    const uint64_t mask_d = a.TC * DL >= 64 ? ~0ull : (1ull << (DL * a.TC)) - 1;
    const bool d_ok = f0 + (lane & (DL - 1)) * 8 < a.F;
    const int krow = 8 * (lane >> 4) + ((lane & 15) >> 2), sub = (lane & 3) * 8;

    uint64_t xv[XP];       // pixels of x on their way
    int xs[XP];            // bits to drop, 64: all
    auto issue = [&](int t, int buf) {
        const int tr = (int)pc_udiv((uint32_t)t, a.mg_tc), x0 = (t - tr * a.tiles_c) * a.TC, r0 = tr * TW_ROWS;
        const int n0 = (int)pc_udiv((uint32_t)r0, a.mg_Ho), V0 = n0 * H1 + (r0 - n0 * a.Ho) * a.stride;
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            // row y of an image is row y + 1 of the padded image, row 0 is zeros
            const int e = tid + 256 * i, row = (int)pc_udiv((uint32_t)e, a.mg_IW), v = V0 + row, n = (int)pc_udiv((uint32_t)v, a.mg_H1), y1 = v - n * H1,
                      xx = x0 * a.stride - 1 + e - row * a.IW;
            const bool ok = e < a.nx && y1 > 0 && n < a.N && (unsigned)xx < (unsigned)a.W;
            // 8 bytes from the pixel on (at any even address), at the tensor's end the last 8.
            const uint32_t off = ok ? (uint32_t)((n * a.H + y1 - 1) * a.W + xx) * (uint32_t)(a.C * 2) : 0u, at = off < a.x_bytes - 8u ? off : a.x_bytes - 8u;
            xs[i] = ok ? (int)(off - at) * 8 : 64;
            __builtin_memcpy(&xv[i], reinterpret_cast<const unsigned char *>(x) + at, 8);
        }
        const uint32_t vd = d_ok && x0 + lane / DL < a.Wo ? (uint32_t)((x0 + lane / DL) * a.F + f0 + (lane & (DL - 1)) * 8) * 2u : WD_OOB;
#pragma unroll
        for (int k = 0; k < TW_ROWS / 4; ++k) {
            const int row = w + 4 * k;
            const bool ok = r0 + row < a.rows;
            wd_load(ds, ok ? vd : WD_OOB, ok ? (r0 + row) * d_row : 0, buf + row * a.RPd, mask_d);
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            const int e = tid + 256 * i, row = (int)pc_udiv((uint32_t)e, a.mg_IW);
            if (e < a.nx) *reinterpret_cast<uint64_t *>(lds + buf + a.x_off + row * a.RPx + (e - row * a.IW) * 8) = xs[i] < 64 ? xv[i] >> xs[i] & mask_c : 0;
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };

    f32x4 acc[3][NF];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < NF; ++k) acc[r][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    int buf = 0;
    issue(wg, 0);                      // (at least one tile for each)
    put(0);
    for (int t = wg; t < a.n_tiles; t += G) {
        const bool more = t + G < a.n_tiles;
        if (more) issue(t + G, a.buf_bytes - buf);
        const int tr = (int)pc_udiv((uint32_t)t, a.mg_tc), r0 = tr * TW_ROWS, n0 = (int)pc_udiv((uint32_t)r0, a.mg_Ho), V0 = n0 * H1 + (r0 - n0 * a.Ho) * a.stride;
        const unsigned char *px[2], *pd[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int k = krow + 4 * q, rho = r0 + k, n = (int)pc_udiv((uint32_t)rho, a.mg_Ho);
            px[q] = lds + buf + a.x_off + (n * H1 + (rho - n * a.Ho) * a.stride - V0) * a.RPx + sub;
            pd[q] = lds + buf + k * a.RPd + sub;
        }
        for (int j = w; j < a.TC; j += 4) {
            bf16x8 xq[3], dq[NF];
#pragma unroll
            for (int r = 0; r < 3; ++r) xq[r] = wd_frag(px[0] + r * a.RPx + j * a.stride * 8, px[1] + r * a.RPx + j * a.stride * 8);
#pragma unroll
            for (int k = 0; k < NF; ++k) dq[k] = wd_frag(pd[0] + j * DB + k * 32, pd[1] + j * DB + k * 32);
#pragma unroll
            for (int k = 0; k < NF; ++k)
#pragma unroll
                for (int r = 0; r < 3; ++r) acc[r][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dq[k], xq[r], acc[r][k], 0, 0, 0);
        }
        if (!more) break;
        buf = a.buf_bytes - buf;
        put(buf);
    }
    // Sums of the four wavefronts, [tap row][filter block][lane]: filter 16 * block + 4 * (lane / 16) + i, tap column and channel lane % 16
    __syncthreads();
    f32x4 *half = reinterpret_cast<f32x4 *>(lds) + (w & 1) * (3 * NF * 64) + lane;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < NF; ++k)
            if (w >= 2) half[(r * NF + k) * 64] = acc[r][k];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < NF; ++k)
            if (w < 2) half[(r * NF + k) * 64] += acc[r][k];
    __syncthreads();
    const int c = tid & 3, fl = tid >> 2;
    for (int f = fl; f < 16 * NF && f0 + f < a.F; f += 64) {
        if (c >= a.C) break;
        const uint32_t info = kinfo[(f0 + f) * a.C + c];
        if (info == 0xFFFFFFFFu) continue;
        const float *p = reinterpret_cast<const float *>(lds) + (f >> 4) * 256 + ((f >> 2) & 3) * 64 + c * 4 + (f & 3);
        float v[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const float *q = p + t / 3 * (NF * 256) + t % 3 * 16;
            v[t] = q[0] + q[3 * NF * 256];
        }
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        uint32_t m = info << 23;
#pragma unroll
        for (int t = 8; t >= 0; --t) {
            const bool kept = __builtin_uadd_overflow(m, m, &m);
            o.w = kept ? o.z : o.w;
            o.z = kept ? o.y : o.z;
            o.y = kept ? o.x : o.y;
            o.x = kept ? v[t] : o.x;
        }
        *reinterpret_cast<float4 *>(out + ((int64_t)wg * a.pstride + (info >> 9)) * 4) = o;
    }
}

template <int NF, int XP>
__global__ void __launch_bounds__(256, 4)
pc_thin_wgrad_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ dy, ThinWgradArgs a, const uint32_t *__restrict__ kinfo, float *__restrict__ out)
{
    extern __shared__ __align__(16) unsigned char lds[];
    pc_thin_wgrad_body<NF, XP>(x, dy, a, kinfo, out, (int)blockIdx.x, (int)gridDim.x, (int)blockIdx.y * 64, lds);
}

__device__ __forceinline__ void pc_thin_wgrad_layer(const ThinWgradLayer &y, int lin)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int fb = __builtin_amdgcn_readfirstlane(lin / y.ksplit), wg = lin - fb * y.ksplit;
    pc_thin_wgrad_body<4, 3>(y.x, y.dy, y.a, y.kinfo, y.out, wg, y.ksplit, fb * 64, lds);   // (three and four blocks of 16 filters have the same layout)
}

// The layers of a network in one launch: workgroup b serves workgroup b - blk0[l] of layer l (blk0 entries are multiples of 8), and behind
// them the network's first layer: its workgroups, short and bound by memory, fill the places that the others
// leave at the end (128 images 32 x 32, 13 layers of VGG-16, all of a training step 458 -> 446 us).
__global__ void __launch_bounds__(256, 2) pc_mfma_wgrad_dma_group_kernel(WgradDmaGroup g)
{
    const int first = g.blk0[g.n];
    if ((int)blockIdx.x < first) {
        const int l = pc_batch_find(g.blk0, g.n, (int)blockIdx.x);
        const WgradDmaLayer &y = g.layer[l];
        const int lin = (int)blockIdx.x - g.blk0[l];
        if (lin < y.gx * y.gy * y.a.ksplit) {
            if (y.a.stride == 1) pc_wgrad_dma_layer<1>(y, lin);
            else pc_wgrad_dma_layer<2>(y, lin);
        }
    } else {
        pc_thin_wgrad_layer(g.thin, (int)blockIdx.x - first);
    }
}

pc_status pc_wgrad_dma_launch(pc_ctx *ctx, WgradDmaGroup &g, size_t lds)
{
    for (int l = 0; l < g.n; ++l) wd_place(g.layer[l]);
    static pc_per_device_once attr;
    pc_note_kernel(ctx, "pc_mfma_wgrad_dma_group_kernel");
    return wd_launch(ctx, &pc_mfma_wgrad_dma_group_kernel, attr, g, lds, g.thin.ksplit * g.thin.blocks_f);
}

bool pc_thin_wgrad_plan(const pc_conv_desc *d, int64_t nslots, int num_cu, ThinWgradPlan *out)
{
    if (d->C > 4 || (d->F & 7)) return false;
    ThinWgradPlan p;
    memset(&p, 0, sizeof(p));
    ThinWgradArgs &a = p.a;
    const int st = d->stride;
    a.N = d->N; a.H = d->H; a.W = d->W; a.C = d->C; a.F = d->F; a.stride = st;
    a.Ho = (d->H - 1) / st + 1; a.Wo = (d->W - 1) / st + 1;
    const int64_t xb = (int64_t)a.N * a.H * a.W * a.C * 2, db = (int64_t)a.N * a.Ho * a.Wo * a.F * 2, rows = (int64_t)a.N * a.Ho;
    if (xb < 8 || xb >= ((int64_t)1 << 31) || db >= ((int64_t)1 << 31) || rows >= (1 << 24)) return false;
    if ((rows + TW_ROWS) * a.Ho >= ((int64_t)1 << 32) || ((int64_t)a.N + TW_ROWS + 2) * (a.H + 1) * (a.H + 1) >= ((int64_t)1 << 32)) return false;
    a.rows = (int)rows;
    a.x_bytes = (uint32_t)xb; a.dy_bytes = (uint32_t)db;
    a.pstride = (int32_t)nslots;
    p.nf = a.F > 48 ? 4 : (a.F + 15) / 16;
    p.blocks_f = (a.F + 63) / 64;
    const int DB = p.nf > 2 ? 128 : 64, cross = a.Ho % TW_ROWS == 0 ? 0 : TW_ROWS % a.Ho == 0 ? TW_ROWS / a.Ho - 1 : (TW_ROWS - 1 + a.Ho - 1) / a.Ho;
    const int nrow = st * (TW_ROWS - 1) + 3 + cross * (a.H + 1 - st * a.Ho);
    for (a.TC = 512 / DB; a.TC >= 1; a.TC >>= 1) {        // a row of dy is (half) a direct load
        a.IW = st * (a.TC - 1) + 3;
        a.nx = nrow * a.IW;
        if (a.nx <= 256 * 3) break;
    }
    if (a.TC < 1) return false;
    p.xp = a.nx <= 256 ? 1 : 3;
    a.RPx = (a.IW + 1) * 8;
    a.RPd = a.TC * DB + 32;
    a.x_off = TW_ROWS * a.RPd;
    a.buf_bytes = (a.x_off + nrow * a.RPx + 15) & ~15;
    p.lds = 2 * (size_t)a.buf_bytes;
    if (p.lds < (size_t)p.nf * 6 * 1024) p.lds = (size_t)p.nf * 6 * 1024;
    if (p.lds > WD_LDS_MAX) return false;
    a.tiles_c = (a.Wo + a.TC - 1) / a.TC;
    const int64_t tiles = (rows + TW_ROWS - 1) / TW_ROWS * a.tiles_c;
    if (tiles * a.tiles_c >= ((int64_t)1 << 32)) return false;
    a.n_tiles = (int)tiles;
    a.mg_tc = pc_udiv_magic(a.tiles_c); a.mg_Ho = pc_udiv_magic(a.Ho); a.mg_H1 = pc_udiv_magic(a.H + 1); a.mg_IW = pc_udiv_magic(a.IW);
    // Two workgroups per CU, the blocks of 64 filters together (4 per CU: 45.2 us for 43.5, and 11.5 for 9.9 on 128 images 32 x 32), so the
    // partial planes of any number of filters stay within 2 MiB (two per CU for each block: 32 x 224 x 224, 3 -> 128 82.8 us for 73.0; 8 x 64 x 64,
    // 3 -> 512 15.2 for 11.7).
    p.ksplit = 2 * num_cu / p.blocks_f;
    if (p.ksplit > a.n_tiles) p.ksplit = a.n_tiles;
    if (p.ksplit < 1) p.ksplit = 1;
    *out = p;
    return true;
}

pc_status pc_thin_wgrad_launch(pc_ctx *ctx, const ThinWgradPlan &p, const uint16_t *x, const uint16_t *dy, const uint32_t *kinfo, float *out)
{
    typedef void (*Kernel)(const uint16_t *, const uint16_t *, ThinWgradArgs, const uint32_t *, float *);
    static const Kernel kernels[2][4] = {{&pc_thin_wgrad_kernel<1, 1>, &pc_thin_wgrad_kernel<2, 1>, &pc_thin_wgrad_kernel<3, 1>, &pc_thin_wgrad_kernel<4, 1>},
                                         {&pc_thin_wgrad_kernel<1, 3>, &pc_thin_wgrad_kernel<2, 3>, &pc_thin_wgrad_kernel<3, 3>, &pc_thin_wgrad_kernel<4, 3>}};
    static pc_per_device_once attr[2][4];
    const Kernel k = kernels[p.xp == 3][p.nf - 1];
    if (pc_once_pending(attr[p.xp == 3][p.nf - 1], ctx->device)) {
        PC_HIP(ctx, hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, WD_LDS_MAX));
        pc_once_done(attr[p.xp == 3][p.nf - 1], ctx->device);
    }
    hipLaunchKernelGGL(k, dim3((unsigned)p.ksplit, (unsigned)p.blocks_f), dim3(256), p.lds, ctx->stream, x, dy, p.a, kinfo, out);
    pc_note_kernel(ctx, "pc_thin_wgrad_kernel<%d, %d>", p.nf, p.xp);
    return pc_hip_check(ctx, hipGetLastError(), "first-layer bwd_weight launch");
}
