// Backward-weight on the matrix cores (bf16 layers), operands straight from NHWC rows in LDS (see pc_wgrad_mfma.hip for the pass
// itself, the splits of the pixels and the partial planes).
#include "pc_wgrad_dma.h"

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

// lin: index of the workgroup in the layer's grid of gx x gy tiles x ksplit splits (x fastest).
template <int ST>
__device__ __forceinline__ void pc_wgrad_dma_body(const uint16_t *__restrict__ x, const uint16_t *__restrict__ dy, const WgradDmaArgs &a,
                                                  const uint32_t *__restrict__ kinfo, float *__restrict__ partial, float *__restrict__ dw, int lin,
                                                  int gx, int gy)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups of an XCD share as few pixel splits as possible (as in pc_mfma_wgrad_ws_body)
    int bx = lin % gx, by = (lin / gx) % gy, bz = lin / (gx * gy);
    {
        const int T = gx * gy, ks = a.ksplit;
        const int xcd = lin & 7, r = lin >> 3;
        int tile = -1;
        if ((ks & 7) == 0) {
            tile = r % T;
            bz = (r / T) * 8 + xcd;
        } else if (ks < 8 && (8 % ks) == 0 && (T % (8 / ks)) == 0) {
            bz = xcd % ks;
            tile = r * (8 / ks) + xcd / ks;
        }
        if (tile >= 0) { bx = tile % gx; by = tile / gx; }
    }
    const int c0 = bx * 64, f0 = by * 64;
    const int fw = w & 1, cw = w >> 1;
    const v4u32 xs = wd_rsrc(x, a.x_bytes), ds = wd_rsrc(dy, a.dy_bytes);
    const int x_row = wd_keep(a.W * a.C * 2), d_row = wd_keep(a.Wo * a.F * 2);       // bytes per row
    const int H1 = wd_keep(a.H + 1), nimg = wd_keep(a.N), rows = wd_keep(a.rows), nrow = wd_keep(a.nrow), TR = wd_keep(a.TR), TC = a.TC, IW = a.IW,
              RPx = wd_keep(a.RPx), RPd = wd_keep(a.RPd), dy_off = a.dy_off, n_ktiles = a.n_ktiles, ksplit = a.ksplit;
    // lanes of the loads of a row: 8 a pixel
    const uint64_t mask_a = IW >= 8 ? ~0ull : (1ull << (8 * IW)) - 1, mask_b = IW > 8 ? ~0ull >> (64 - 8 * (IW - 8)) : 0,
                   mask_d = TC >= 8 ? ~0ull : (1ull << (8 * TC)) - 1;
    const bool x_ok = c0 + (lane & 7) * 8 < a.C, d_ok = f0 + (lane & 7) * 8 < a.F;
    // where this lane's transposing reads start inside 4 pixels' rows (4 of 16 channels or filters), and the first row it reads
    // (stride 2: the 32 reduction entries are 16 rows of two columns that follow each other, for less LDS per tile)
    constexpr int KROWS = ST == 1 ? 32 : 16;
    const int sub = (lane & 3) * 8, krow = 8 * ((lane >> 4) & (KROWS / 8 - 1)) + ((lane & 15) >> 2), kcol = ST == 1 ? 0 : lane >> 5;

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
            // a wavefront's load brings 8 pixels of a row, the x columns past the 8th come in a second one
            const int col = lane >> 3;
            uint32_t vx[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int xx = x0 * ST - 1 + p * 8 + col;
                vx[p] = x_ok && (unsigned)xx < (unsigned)a.W ? (uint32_t)(xx * a.C + c0 + (lane & 7) * 8) * 2u : WD_OOB;
            }
            const uint32_t vd = d_ok && x0 + col < a.Wo ? (uint32_t)((x0 + col) * a.F + f0 + (lane & 7) * 8) * 2u : WD_OOB;
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
        for (int hh = 0; hh < TR; hh += KROWS) {
            const unsigned char *pr[3][2], *pd[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int k = hh + krow + 4 * q, rho = r0 + k, n = (int)pc_udiv((uint32_t)rho, a.mg_Ho);
                pr[0][q] = lds + (n * H1 + (rho - n * a.Ho) * ST - V0) * RPx + cw * 64 + sub + kcol * (ST * 128);
                pr[1][q] = pr[0][q] + RPx;
                pr[2][q] = pr[1][q] + RPx;
                pd[q] = lds + dy_off + k * RPd + fw * 64 + sub + kcol * 128;
            }
            bf16x8 xq[3][2], dq[4][2];
            auto read_x = [&](int r, int h, int col) __attribute__((always_inline)) { xq[r][h] = wd_frag(pr[r][0] + col * 128 + h * 32, pr[r][1] + col * 128 + h * 32); };
            auto read_d = [&](int col) __attribute__((always_inline)) {
#pragma unroll
                for (int h = 0; h < 2; ++h) dq[col & 3][h] = wd_frag(pd[0] + col * 128 + h * 32, pd[1] + col * 128 + h * 32);
            };
            read_d(0);
#pragma unroll
            for (int i = 0; i < 6; ++i) read_x(i >> 1, i & 1, 0);
            if constexpr (ST == 2) {
                // pairs of output columns: tap column q of the pair from column c is the pair of x columns 2c + q and 2c + q + 2
#pragma unroll
                for (int u = 0; u < 9; ++u) {
                    const int c = 2 * (u / 3), q = u % 3;
                    if (c < TC) {
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
            constexpr int LAST = 9;              // last x column of a tile of 8
#pragma unroll
            for (int X = 0; X <= LAST; ++X) {
                if (X < IW) {
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
                        if (j < TC) {
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
    // Epilogue: a lane holds all nine taps of its 16 kernels; the 4 kept ones of a kept kernel move down in place and are written in
    // compact slot order. (Tap by tap from the last: a kept one becomes the first of the kept values and moves the others up.)
    float *pout = a.ksplit > 1 ? partial + (int64_t)bz * a.pstride * 4 : dw;
    uint32_t info[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int f = f0 + fw * 32 + (k >> 3) * 16 + 4 * (lane >> 4) + (k & 3), c = c0 + cw * 32 + ((k >> 2) & 1) * 16 + (lane & 15);
        info[k] = f < a.F && c < a.C ? kinfo[(int64_t)f * a.C + c] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int t = 8; t >= 0; --t) {
            const bool kept = info[k] >> t & 1u;
            o.w = kept ? o.z : o.w;
            o.z = kept ? o.y : o.z;
            o.y = kept ? o.x : o.y;
            o.x = kept ? acc[t][k >> 3][(k >> 2) & 1][k & 3] : o.x;
        }
        if (info[k] != 0xFFFFFFFFu) *reinterpret_cast<float4 *>(pout + (int64_t)(info[k] >> 9) * 4) = o;
    }
}

// The layers of a network in one launch: workgroup b serves workgroup b - blk0[l] of layer l (blk0 entries are multiples of 8).
__global__ void __launch_bounds__(256, 2) pc_mfma_wgrad_dma_kernel(WgradDmaGroup g)
{
    const int l = pc_batch_find(g.blk0, g.n, (int)blockIdx.x);
    const WgradDmaLayer &y = g.layer[l];
    const int lin = (int)blockIdx.x - g.blk0[l];
    if (lin >= y.gx * y.gy * y.a.ksplit) return;
    if (y.a.stride == 1) pc_wgrad_dma_body<1>(y.x, y.dy, y.a, y.kinfo, y.partial, y.dw, lin, y.gx, y.gy);
    else pc_wgrad_dma_body<2>(y.x, y.dy, y.a, y.kinfo, y.partial, y.dw, lin, y.gx, y.gy);
}

bool pc_wgrad_dma_plan(const pc_conv_desc *d, int64_t nslots, WgradDmaArgs *out, int *ct, int *ft, size_t *lds, double *tile_us)
{
    WgradDmaArgs a;
    memset(&a, 0, sizeof(a));
    const int st = d->stride;
    if ((d->C & 7) || (d->F & 7)) return false;
    a.N = d->N; a.H = d->H; a.W = d->W; a.C = d->C; a.F = d->F; a.stride = st;
    a.Ho = (d->H - 1) / st + 1; a.Wo = (d->W - 1) / st + 1;
    const int64_t xb = (int64_t)a.N * a.H * a.W * a.C * 2, db = (int64_t)a.N * a.Ho * a.Wo * a.F * 2, rows = (int64_t)a.N * a.Ho;
    if (xb >= ((int64_t)1 << 31) || db >= ((int64_t)1 << 31) || rows >= (1 << 24)) return false;
    a.x_bytes = (uint32_t)xb; a.dy_bytes = (uint32_t)db;
    a.rows = (int)rows;
    double best = -1.0;
    const int krows = st == 1 ? 32 : 16, cstep = st;      // rows and columns of a step
    for (int TR = krows; TR <= 64; TR += krows)
        for (int tcn = cstep; tcn <= (st == 1 ? 8 : 6) && tcn < a.Wo + cstep; tcn += cstep)
            for (int pad = 32; pad >= 0; pad -= 32) {
                // image boundaries inside a tile (tiles start at multiples of TR); rows past the last image lie as if more images followed
                const int cross = a.Ho % TR == 0 ? 0 : TR % a.Ho == 0 ? TR / a.Ho - 1 : (TR - 1 + a.Ho - 1) / a.Ho;
                const int nrow = st * (TR - 1) + 3 + cross * (a.H + 1 - st * a.Ho);
                const int IW = st * (tcn - 1) + 3, RPx = IW * 128 + (st == 1 ? 32 : 16), RPd = tcn * 128 + pad;
                // columns of dy that are read past the end of a row: three, none past the eighth (stride 1), or the next pair (stride 2)
                const int past = st == 1 ? (tcn + 3 < 8 ? 3 : 8 - tcn) : tcn < 6 ? 2 : 0, room = past * 128 > pad ? past * 128 - pad : 0;
                if (nrow * RPx + TR * RPd + room > WD_LDS_MAX) continue;
                const int tc_n = (a.Wo + tcn - 1) / tcn, tr_n = (int)((rows + TR - 1) / TR);
                const double fill = (double)rows * a.Wo / ((double)tr_n * TR * tc_n * tcn);
                const double mfma = TR / 32.0 * tcn * 36 * 16, load = ((double)nrow * IW + (double)TR * tcn) * 128 / 30.0;   // cycles
                const double eff = fill * mfma / ((mfma > load ? mfma : load) + 300 + 150.0 * (TR / 16));
                if (eff > best) {
                    best = eff;
                    a.TR = TR; a.TC = tcn; a.IW = IW; a.nrow = nrow; a.RPx = RPx; a.RPd = RPd; a.dy_off = nrow * RPx;
                    a.tiles_c = tc_n; a.n_ktiles = tr_n * tc_n;
                    *lds = (size_t)(nrow * RPx + TR * RPd + room);
                }
            }
    if (best < 0.0) return false;
    if ((rows + 64) * a.Ho >= ((int64_t)1 << 32) || ((int64_t)a.N + 66) * (a.H + 1) * (a.H + 1) >= ((int64_t)1 << 32) ||
        (int64_t)a.n_ktiles * a.tiles_c >= ((int64_t)1 << 32)) return false;
    a.pstride = (int32_t)nslots;
    a.mg_tc = pc_udiv_magic(a.tiles_c); a.mg_Ho = pc_udiv_magic(a.Ho); a.mg_H1 = pc_udiv_magic(a.H + 1);
    *tile_us = 0.55 * (a.TR / krows) * (a.TC / cstep) + 1.3;
    *ct = (a.C + 63) / 64;
    *ft = (a.F + 63) / 64;
    *out = a;
    return true;
}

pc_status pc_wgrad_dma_launch(pc_ctx *ctx, const WgradDmaGroup &g, size_t lds)
{
    static pc_per_device_once attr;
    if (pc_once_pending(attr, ctx->device)) {
        PC_HIP(ctx, hipFuncSetAttribute((const void *)pc_mfma_wgrad_dma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, WD_LDS_MAX));
        pc_once_done(attr, ctx->device);
    }
    hipLaunchKernelGGL(pc_mfma_wgrad_dma_kernel, dim3((unsigned)g.blk0[g.n]), dim3(256), lds, ctx->stream, g);
    pc_note_kernel(ctx, "pc_mfma_wgrad_dma_kernel");
    return pc_hip_check(ctx, hipGetLastError(), "MFMA bwd_weight (direct loads) launch");
}
