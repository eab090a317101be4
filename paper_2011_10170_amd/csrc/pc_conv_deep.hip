// Forward / backward-data of layers with few pixels and many reduction channels (see pc_mfma.h and pc_conv_mfma.hip for the operand tiles).
#include "pc_dma.h"

#include <math.h>
#include <algorithm>

// What bounds such a layer (one 14 x 14 image, 512 -> 512: 4.7 MB of weights for 0.9 GFLOP) is how its weights come: tiles that walk the reduction
// a chunk after the other ask a CU for 300 to 600 KB in a dozen round trips. Here a workgroup of 8 wavefronts owns 16 * MF output channels x
// 16 * NF pixels, the wavefronts share out the chunks of 32 reduction channels, and everything is asked for at once: a
// wavefront's weights, one or two chunks, straight into registers in operand order, and the pixels that the tile touches, all channels, by direct
// loads. One memory round trip, up to 144 matrix instructions a wavefront from LDS, and the eight partial tiles are added through LDS in
// wavefront order.
//   Pixels: those of a tile follow each other in raster order over rows and images, so what they touch is one range of memory, 16 * NF + 2 * W + 2
//     pixels, and a neighbour is a constant away. One that lies outside the map is read from a zero in LDS instead.
//   LDS: pixels lie as in memory, but the 16-byte pieces of a pixel in an order turned by its number (the direct load of a lane asks for
//     another piece), or 16 pixels' operands would stand in the same banks.
// One 14 x 14 image, 512 -> 512 7.8 us (the register kernel) -> 5.3, 128 images 2 x 2 8.4 -> 6.7, 8 x 6 x 6 images 168 -> 512 6.1 -> 5.0; of 440 passes of 16 to
// 4096 pixels it is the fastest on 338, by 1.15 on average. What bounds it now: a CU takes 65 to 70 KB a microsecond, of which a tile
// of 16 channels x 32 pixels asks for 209 KB at 512 channels (a tile of 32 x 64 for 389: 8.6 us). Addresses are made while the loads are on their way
// (between the matrix instructions: 7.4 us).
struct DeepArgs {
    int32_t P, W, H, in_CH, out_CH;  // pixels of all images, the map
    int32_t KS, nch, flip;           // k-steps of 16 per tap in the operand tiles; chunks of 32 reduction channels
    int32_t CP, mask, loads, zero;   // 16-byte pieces of a pixel, those whose order turns less 1, direct loads per wavefront, LDS offset of the zero
    int32_t count, p_tiles;          // staged pixels, tiles of pixels
    uint32_t mg_CP, mg_W, mg_H, mg_pt;
    uint32_t in_bytes, out_bytes, wz_bytes;
    const uint16_t *act_mask;
};

template <int MF, int NF, int NC, int ACT>
__global__ void __launch_bounds__(512, 2)
pc_mfma_conv_deep_kernel(const uint16_t *__restrict__ in, uint16_t *__restrict__ out, const uint16_t *__restrict__ wz, DeepArgs g)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63, kg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups that share weights share an XCD
    const int G = gridDim.x, b = blockIdx.x, vb = (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
    const int mt = (int)pc_udiv((uint32_t)vb, g.mg_pt), p0 = (vb - mt * g.p_tiles) * (16 * NF), m0 = mt * (16 * MF);

    // weights of this wavefront's chunks, w and w + 8 (past the last: zeros)
    const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wz), 0, g.wz_bytes, 0x00020000);
    const int wvo = (kg >> 1) * 1024 + (kg & 1) * 512 + (lane & 15) * 16;
    bf16x8 A[NC][9][MF];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int a = 0; a < MF; ++a) {
                const int row = m0 + 16 * a, ch = w + 8 * c;
                const v4u32 v = __builtin_amdgcn_raw_buffer_load_b128(wsrc, ch < g.nch ? wvo : (int)DM_OOB, (((row >> 5) * 9 + (g.flip ? 8 - t : t)) * g.KS + ch * 2) * 1024 + (row & 16) * 16, 0);
                __builtin_memcpy(&A[c][t][a], &v, 16);
            }
    // the tile's pixels and their neighbours, staged pixel q is p0 - W - 1 + q
    const v4u32 xs = dm_rsrc(in, g.in_bytes);
    for (int i = 0; i < g.loads; ++i) {
        const uint32_t e = (uint32_t)((i * 8 + w) * 64 + lane), q = pc_udiv(e, g.mg_CP), j = e - q * g.CP;
        const int p = p0 - g.W - 1 + (int)q;
        const bool ok = (int)q < g.count && (unsigned)p < (unsigned)g.P;
        dm_load(xs, (int)(ok ? ((uint32_t)p * g.CP + (j ^ (q & g.mask))) * 16u : DM_OOB), 0, (i * 8 + w) * 1024);
    }
    if (threadIdx.x < 256) *reinterpret_cast<uint32_t *>(lds + g.zero + threadIdx.x * 4) = 0u;
    // where the sums of this thread go, and the mask of the fused step
    const __amdgpu_buffer_rsrc_t osrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, g.out_bytes, 0x00020000);
    const int px = (int)threadIdx.x / (4 * MF), c4 = (int)threadIdx.x % (4 * MF), om = m0 + 4 * c4;
    const bool mine = px < 16 * NF && p0 + px < g.P && om < g.out_CH;
    const uint32_t off = mine ? ((uint32_t)(p0 + px) * (uint32_t)g.out_CH + (uint32_t)om) * 2u : DM_OOB;
    v2u32 mk = {0u, 0u};
    if (ACT == PC_ACT_RELU_MASK)
        mk = __builtin_amdgcn_raw_buffer_load_b64(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.act_mask), 0, g.out_bytes, 0x00020000), (int)off, 0, 0);
    // where this lane reads the operands of chunk w; those of chunk w + 8 are 32 pieces further, whose order turns alike
    // (channels past the last: zeros)
    const int first = w * 4 + kg;
    const bool more = first + 32 < g.CP;
    int at[9][NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const uint32_t p = (uint32_t)(p0 + 16 * f + (lane & 15)), r = pc_udiv(p, g.mg_W), x = p - r * g.W, y = r - pc_udiv(r, g.mg_H) * g.H;
        const bool on = (int)p < g.P && first < g.CP, cols[3] = {x > 0, true, (int)x < g.W - 1}, rows[3] = {y > 0 && on, on, (int)y < g.H - 1 && on};
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int q = 16 * f + (lane & 15) + t / 3 * g.W + t % 3, in_lds = q * (g.CP * 16) + ((first ^ (q & g.mask)) << 4);
            at[t][f] = rows[t / 3] && cols[t % 3] ? in_lds : g.zero;
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    f32x4 acc[MF][NF];
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[a][f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            bf16x8 B[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) B[f] = *reinterpret_cast<const bf16x8 *>(lds + (c == 0 ? at[t][f] : more ? at[t][f] + 512 : g.zero));
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int a = 0; a < MF; ++a) acc[a][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[c][t][a], B[f], acc[a][f], 0, 0, 0);
        }
    }
    // partial tiles [wavefront][pixel][4 channels], a pixel's in an order turned by its number
    __syncthreads();
    float4 *red = reinterpret_cast<float4 *>(lds);
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
        for (int f = 0; f < NF; ++f)
            red[(w * (16 * NF) + 16 * f + (lane & 15)) * (4 * MF) + ((4 * a + kg) ^ (lane & (4 * MF - 1)))] = make_float4(acc[a][f][0], acc[a][f][1], acc[a][f][2], acc[a][f][3]);
    __syncthreads();
    if (px >= 16 * NF) return;
    float4 s = red[px * (4 * MF) + (c4 ^ (px & (4 * MF - 1)))];
#pragma unroll
    for (int k = 1; k < 8; ++k) {
        const float4 v = red[(k * (16 * NF) + px) * (4 * MF) + (c4 ^ (px & (4 * MF - 1)))];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    v2u32 o = {pc_pack_bf16x2(s.x, s.y), pc_pack_bf16x2(s.z, s.w)};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (ACT == PC_ACT_RELU) o[k] = pc_relu_bf16x2(o[k]);
        if (ACT == PC_ACT_RELU_MASK) o[k] = pc_mask_bf16x2(o[k], mk[k]);
    }
    __builtin_amdgcn_raw_buffer_store_b64(o, osrc, (int)off, 0, 0);
}

// ---- plan and launch
#define DP_LDS_MAX (160 * 1024)
struct DeepCand { int code, mf, nf; };
static const DeepCand kDeep[] = {{51, 1, 2}, {52, 1, 4}, {53, 2, 2}, {54, 2, 4}};
constexpr int kNumDeep = sizeof(kDeep) / sizeof(kDeep[0]);

static bool plan_deep(const MfmaArgs &g, bool flip, const DeepCand &c, DeepArgs *out, size_t *lds, int *grid, double *est, double *least, int num_cu)
{
    DeepArgs t;
    memset(&t, 0, sizeof(t));
    const int64_t P = (int64_t)g.N * g.in_H * g.in_W, in_bytes = P * g.in_CH * 2, out_bytes = P * g.out_CH * 2;
    if (P >= (1 << 20) || in_bytes >= ((int64_t)1 << 31) || out_bytes >= ((int64_t)1 << 31)) return false;
    t.P = (int)P; t.W = g.in_W; t.H = g.in_H; t.in_CH = g.in_CH; t.out_CH = g.out_CH;
    if (P * t.W >= ((int64_t)1 << 32) || P * t.H >= ((int64_t)1 << 32)) return false;     // multiply-high divisions stay exact
    t.KS = g.KS; t.flip = flip;
    t.nch = (g.in_CH + 31) / 32;
    t.CP = g.in_CH / 8;
    t.mask = std::min(t.CP & -t.CP, 16) - 1;
    t.count = 16 * c.nf + 2 * t.W + 2;
    if ((int64_t)t.count * t.CP * 16 > DP_LDS_MAX) return false;
    t.loads = (t.count * t.CP + 511) / 512;
    t.zero = t.loads * 8192;
    *lds = std::max((size_t)t.zero + 1024, (size_t)8 * 16 * c.nf * 16 * c.mf * 4);
    if (*lds > DP_LDS_MAX) return false;
    t.p_tiles = ((int)P + 16 * c.nf - 1) / (16 * c.nf);
    const int m_tiles = (g.out_CH + 16 * c.mf - 1) / (16 * c.mf);
    if ((int64_t)m_tiles * t.p_tiles * t.p_tiles >= ((int64_t)1 << 32)) return false;
    *grid = m_tiles * t.p_tiles;
    t.mg_CP = pc_udiv_magic(t.CP); t.mg_W = pc_udiv_magic(t.W); t.mg_H = pc_udiv_magic(t.H); t.mg_pt = pc_udiv_magic(t.p_tiles);
    t.in_bytes = (uint32_t)in_bytes; t.out_bytes = (uint32_t)out_bytes;
    t.wz_bytes = (uint32_t)((size_t)((g.out_CH + 127) / 128 * 4) * 9 * t.KS * 1024);
    t.act_mask = g.act_mask;
    // Estimated time (us): a start, a round trip for every set of workgroups that the CUs hold at once (one or two each, by LDS and registers), and
    // the staging and the matrix instructions of what a CU gets (1760 timings of 440 passes, 5 % rms; among the four 1.4 % behind the best)
    const bool two = t.nch > 8;
    int occ = (int)(DP_LDS_MAX / *lds);
    occ = std::min(occ, c.mf * c.nf <= (two ? 2 : 4) ? 2 : 1);
    const double n = (double)*grid / num_cu, share = std::max(1.0, 0.5 * (ceil(n) + n));
    *est = 2.89 + ceil(n / occ) * (two ? 1.42 : 1.01) + share * (0.0166 * t.count * t.CP / 64.0 + 0.0217 * 9.0 * c.mf * c.nf * (two ? 2 : 1));
    // Those timings are of up to 4096 pixels. Several tiles per CU wait for LDS and for memory: 15 % below a fit to 2400 timings of 4 to 2000000 pixels is
    // the estimate where it is the larger one (112 x 31 x 28, 496 -> 16: 47.9 us in tiles of 16 x 64, 32 by the line above, 31.0 by the kernel for direct
    // loads; 65 x 22 x 20, 440 -> 32 18.6, 14.0). Of 7522 passes of drawn layers and networks it sends 23 to another kernel: 1.03 times as fast among
    // themselves, 1.08 between passes of other weights and tensors; the worst 8 % slower (11 x 12 x 12, 512 -> 256 9.2 -> 9.9 us).
    const double work = (two ? 0.861 * ceil(n / occ) : 0.0) + share * (0.0115 * t.count * t.CP / 64.0 + 0.0376 * 9.0 * c.mf * c.nf * (two ? 2 : 1));
    const double moved = 0.0568e-6 * ((double)t.p_tiles * t.count * t.CP * 16.0 + (double)out_bytes) + 0.0069e-6 * *grid * (t.count * t.CP * 16.0 + 288.0 * c.mf * g.in_CH);
    *least = 2.14 + pow(pow(work, 1.5) + pow(moved, 1.5), 1.0 / 1.5);
    *out = t;
    return true;
}

typedef void (*DeepKernel)(const uint16_t *, uint16_t *, const uint16_t *, DeepArgs);
#define DP_ACTS(MF, NF, NC) {&pc_mfma_conv_deep_kernel<MF, NF, NC, PC_ACT_NONE>, &pc_mfma_conv_deep_kernel<MF, NF, NC, PC_ACT_RELU>, &pc_mfma_conv_deep_kernel<MF, NF, NC, PC_ACT_RELU_MASK>}
#define DP_UNITS(MF, NF) {DP_ACTS(MF, NF, 1), DP_ACTS(MF, NF, 2)}
static const DeepKernel kDeepKernels[kNumDeep][2][3] = {DP_UNITS(1, 2), DP_UNITS(1, 4), DP_UNITS(2, 2), DP_UNITS(2, 4)};
#undef DP_UNITS
#undef DP_ACTS

// pcfg: -1 or a code of kDeep. *launched stays 0 where the kernel does not take the launch or no estimate is below limit (us).
pc_status pc_run_mfma_conv_deep(pc_ctx *ctx, int pcfg, double limit, const MfmaArgs &g, bool flip, const uint16_t *in, uint16_t *out,
                                const uint16_t *wz, int *launched, double *us, int act)
{
    *launched = 0;
    if (g.lstep != 1 || g.oscale != 1 || (g.in_CH & 7) || g.in_CH > 512 || (g.out_CH & 7) || !pc_direct_loads(in)) return PC_OK;
    DeepArgs best;
    size_t best_lds = 0;
    int best_grid = 0, best_k = -1;
    double best_est = limit, best_least = 0.0;
    for (int k = 0; k < kNumDeep; ++k) {
        if (pcfg >= 0 && pcfg != kDeep[k].code) continue;
        DeepArgs t;
        size_t lds;
        int grid;
        double est, least;
        if (!plan_deep(g, flip, kDeep[k], &t, &lds, &grid, &est, &least, ctx->num_cu)) continue;
        if (pcfg >= 0 || est < best_est) { best = t; best_lds = lds; best_grid = grid; best_k = k; best_est = est; best_least = least; }
    }
    best_est = std::max(best_est, best_least);
    if (best_k < 0 || (pcfg < 0 && best_est >= limit)) return PC_OK;
    if (us) {                        // only asked for
        *us = best_est;
        *launched = kDeep[best_k].code;
        return PC_OK;
    }
    const int nc = best.nch > 8;
    const DeepKernel kernel = kDeepKernels[best_k][nc][act];
    static pc_per_device_once attr[kNumDeep][2][3];
    if (pc_once_pending(attr[best_k][nc][act], ctx->device)) {
        PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, DP_LDS_MAX));
        pc_once_done(attr[best_k][nc][act], ctx->device);
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)best_grid), dim3(512), best_lds, ctx->stream, in, out, wz, best);
    *launched = kDeep[best_k].code;
    pc_note_kernel(ctx, "pc_mfma_conv_deep_kernel<%d, %d, %d, %d>", kDeep[best_k].mf, kDeep[best_k].nf, 1 + nc, act);
    return pc_hip_check(ctx, hipGetLastError(), "MFMA conv (deep) launch");
}
