// Backward-weight of layers with few pixels in one launch (see pc_wgrad_dma.hip for the operands by transposing LDS reads).
#include "pc_dma.h"

#include <math.h>
#include <algorithm>

// Where the pixels are few, splitting them over workgroups costs more than it gains: partial planes are written, and a second launch adds them.
// Here a workgroup of 8 wavefronts owns 16 * MF filters x 16 * MC channels of all nine taps and walks all pixels; the wavefronts take groups of
// 32 pixels in turn, their sums are added in LDS in wavefront order and the kept taps leave in compact order. No scratch is needed. Launch by
// launch 1 image 14 x 14, 512 -> 512: 12.3 -> 7.9 us; 4 images 14 x 14, 256 -> 256: 12.4 -> 6.0; in a graph 3 images 27 x 27, 24 -> 64:
// 10.3 -> 7.5. (Against 64 bits its error is 0.91 to 1.23 times that of split pixels, 1.06 on average of 17 drawn layers, 2e-8 to 1e-7 both: float32 sums in
// another order.) Bound by a start (3 us) and then by the serial chain of one workgroup: 5000 pixels 96 -> 304 16.5 us, the pixels split 14.5.
//   Cells: x and dy are staged as the map with one zero column after every row and one zero row after every image (the direct loads of
//     those lanes lie outside the tensor), so that a tap is a constant distance and nothing is masked: a zero of dy adds nothing.
//   LDS: [block of 16 channels][cell][16]; a transposing read takes 4 cells of 16 channels from 128 bytes, and the 32 cells of a step are dealt to
//     the lanes so that the four groups of 16 lanes read 512 bytes side by side.
struct FewWgradArgs {
    int32_t N, H, W, C, F;
    int32_t R, I;                    // cells of a row and of an image
    int32_t cells, xcells, chunks;   // of a chunk: cells of dy (a multiple of 32) and of x (rounded up to one)
    int32_t tiles_c;
    uint32_t mg_R, mg_I, mg_tc;
    uint32_t x_bytes, dy_bytes;
};

template <int MF, int MC>
__global__ void __launch_bounds__(512, 2)
pc_mfma_wgrad_dma_few_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ dy, FewWgradArgs a, const uint32_t *__restrict__ kinfo,
                             float4 *__restrict__ dw)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int COPIES = MF * MC == 4 ? 4 : 8, UNITS = 9 * MF * MC, KERNELS = 256 * MF * MC, PER = (KERNELS + 511) / 512;
    const int lane = threadIdx.x & 63, h = lane >> 4, i16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = gridDim.x, b = blockIdx.x, vb = (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
    const int tf = (int)pc_udiv((uint32_t)vb, a.mg_tc), f0 = tf * (16 * MF), c0 = (vb - tf * a.tiles_c) * (16 * MC);
    // (compact slot, pattern mask) of the kernels that this thread writes at the end
    uint32_t info[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int id = k * 512 + (int)threadIdx.x, f = f0 + id / (16 * MC), c = c0 + id % (16 * MC);
        const bool on = id < KERNELS && f < a.F && c < a.C;
        info[k] = kinfo[on ? f * a.C + c : 0];
        if (!on) info[k] = 0xFFFFFFFFu;
    }
    const v4u32 xs = dm_rsrc(x, a.x_bytes), ds = dm_rsrc(dy, a.dy_bytes);
    const int x_at = MF * a.cells * 32;
    // 32 cells of every block of 16 channels from cell v on, 16 bytes per lane
    auto stage = [&](const v4u32 &rsrc, int blocks, int CH, int ch0, int v, int at, int block_bytes) __attribute__((always_inline)) {
        const int u = v + (lane >> 1), n = (int)pc_udiv((uint32_t)(u < 0 ? 0 : u), a.mg_I), rem = u - n * a.I, y = (int)pc_udiv((uint32_t)(rem < 0 ? 0 : rem), a.mg_R), xx = rem - y * a.R;
        const bool ok = u >= 0 && n < a.N && y < a.H && xx < a.W;
        const uint32_t off = ((uint32_t)((n * a.H + y) * a.W + xx) * (uint32_t)CH + (uint32_t)(ch0 + (lane & 1) * 8)) * 2u;
        for (int k = 0; k < blocks; ++k)
            dm_load(rsrc, (int)(ok && ch0 + k * 16 + (lane & 1) * 8 < CH ? off : DM_OOB), k * 32, at + k * block_bytes);
    };
    f32x4 acc[9][MF][MC];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int f = 0; f < MF; ++f)
#pragma unroll
            for (int c = 0; c < MC; ++c) acc[t][f][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    typedef short i16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) i16x4 *lds4;
    auto operand = [&](int at) __attribute__((always_inline)) -> bf16x8 {       // cells 4h .. 4h + 3 and 16 + 4h .. of a step, channel i16
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(lds + at)), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(lds + at + 512));
        const short __attribute__((ext_vector_type(8))) v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        bf16x8 r;
        __builtin_memcpy(&r, &v, 16);
        return r;
    };
    const int mine = (4 * h + (i16 >> 2)) * 32 + (i16 & 3) * 8;
    for (int q = 0; q < a.chunks; ++q) {
        const int v0 = q * a.cells;
        if (q) __syncthreads();               // every wavefront has read what the loads replace
        for (int k = w; k < a.cells >> 5; k += 8) stage(ds, MF, a.F, f0, v0 + k * 32, k * 1024, a.cells * 32);
        for (int k = w; k < a.xcells >> 5; k += 8) stage(xs, MC, a.C, c0, v0 + k * 32 - a.R - 1, x_at + k * 1024, a.xcells * 32);
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        for (int k = w; k < a.cells >> 5; k += 8) {
            bf16x8 A[MF];
#pragma unroll
            for (int f = 0; f < MF; ++f) A[f] = operand(mine + k * 1024 + f * a.cells * 32);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                bf16x8 B[MC];
#pragma unroll
                for (int c = 0; c < MC; ++c) B[c] = operand(mine + x_at + k * 1024 + (t / 3 * a.R + t % 3) * 32 + c * a.xcells * 32);
#pragma unroll
                for (int f = 0; f < MF; ++f)
#pragma unroll
                    for (int c = 0; c < MC; ++c) acc[t][f][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[f], B[c], acc[t][f][c], 0, 0, 0);
            }
        }
    }
    // Sums of the wavefronts: [wavefront][tap, block of filters, block of channels][lane][4 filters], added by units; of eight large ones the upper
    // half is added to the lower first.
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);
    auto unit = [&](int u) __attribute__((always_inline)) -> f32x4 & { return acc[u / (MF * MC)][u / MC % MF][u % MC]; };
    __syncthreads();
    if constexpr (COPIES == 4) {
        if (w >= 4) {
#pragma unroll
            for (int u = 0; u < UNITS; ++u) red[((w - 4) * UNITS + u) * 64 + lane] = unit(u);
        }
        __syncthreads();
        if (w < 4) {
#pragma unroll
            for (int u = 0; u < UNITS; ++u) unit(u) += red[(w * UNITS + u) * 64 + lane];
#pragma unroll
            for (int u = 0; u < UNITS; ++u) red[(w * UNITS + u) * 64 + lane] = unit(u);      // (what this wavefront has read itself)
        }
    } else {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) red[(w * UNITS + u) * 64 + lane] = unit(u);
    }
    __syncthreads();
    for (int u = w; u < UNITS; u += 8) {
        f32x4 s = red[u * 64 + lane];
#pragma unroll
        for (int k = 1; k < COPIES; ++k) s += red[(k * UNITS + u) * 64 + lane];
        red[u * 64 + lane] = s;               // (read by this wavefront alone)
    }
    __syncthreads();
    const float *sum = reinterpret_cast<const float *>(lds);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (info[k] == 0xFFFFFFFFu) continue;
        const int id = k * 512 + (int)threadIdx.x, f = id / (16 * MC), c = id % (16 * MC);
        const int at = ((f >> 4) * MC + (c >> 4)) * 256 + ((((f & 15) >> 2) * 16 + (c & 15)) * 4) + (f & 3);
        uint32_t left = info[k] & 511u;
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j, left &= left - 1u) v[j] = sum[(__ffs((int)left) - 1) * (MF * MC * 256) + at];
        dw[info[k] >> 9] = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// ---- plan and launch
#define FW_LDS_MAX (160 * 1024)
struct FewCand { int mf, mc; };
static const FewCand kFew[] = {{1, 1}, {1, 2}, {2, 1}, {2, 2}};
typedef void (*FewKernel)(const uint16_t *, const uint16_t *, FewWgradArgs, const uint32_t *, float4 *);
static const FewKernel kFewKernels[] = {&pc_mfma_wgrad_dma_few_kernel<1, 1>, &pc_mfma_wgrad_dma_few_kernel<1, 2>, &pc_mfma_wgrad_dma_few_kernel<2, 1>, &pc_mfma_wgrad_dma_few_kernel<2, 2>};

static bool plan_few(const pc_conv_desc *d, const FewCand &c, int num_cu, FewWgradArgs *out, size_t *lds, int *grid, double *est)
{
    FewWgradArgs a;
    memset(&a, 0, sizeof(a));
    a.N = d->N; a.H = d->H; a.W = d->W; a.C = d->C; a.F = d->F;
    a.R = d->W + 1;
    const int64_t I = (int64_t)(d->H + 1) * a.R, cells = I * d->N, px = (int64_t)d->N * d->H * d->W;
    if (cells > (1 << 20) || px * d->C * 2 >= ((int64_t)1 << 31) || px * d->F * 2 >= ((int64_t)1 << 31)) return false;
    a.I = (int32_t)I;
    if ((cells + 8192) * a.I >= ((int64_t)1 << 32)) return false;       // multiply-high divisions stay exact
    const int halo = (2 * a.R + 2 + 31) / 32 * 32;
    const int most = (FW_LDS_MAX / 32 - c.mc * halo) / (c.mf + c.mc) / 32 * 32;
    if (most < 256) return false;
    a.chunks = (int)((cells + most - 1) / most);
    a.cells = (int)(((cells + a.chunks - 1) / a.chunks + 31) / 32 * 32);
    a.xcells = a.cells + halo;
    const int copies = c.mf * c.mc == 4 ? 4 : 8;
    *lds = std::max((size_t)(c.mf * a.cells + c.mc * a.xcells) * 32, (size_t)copies * 9 * c.mf * c.mc * 1024);
    a.tiles_c = (d->C + 16 * c.mc - 1) / (16 * c.mc);
    *grid = a.tiles_c * ((d->F + 16 * c.mf - 1) / (16 * c.mf));
    if ((int64_t)*grid * a.tiles_c >= ((int64_t)1 << 32)) return false;
    a.mg_R = pc_udiv_magic(a.R); a.mg_I = pc_udiv_magic(a.I); a.mg_tc = pc_udiv_magic(a.tiles_c);
    a.x_bytes = (uint32_t)(px * d->C * 2); a.dy_bytes = (uint32_t)(px * d->F * 2);
    // Estimated time (us): a start, of every chunk a wait, its loads and its products (as LDS reads of a wavefront), workgroups that share a CU,
    // the bytes staged by all, the sums of the wavefronts. Fitted to 900 timings of 230 layers (6 % rms); on the 133 layers
    // of profiles/wgrad_few_timings_bf16.csv that come here the tile taken is 0.7 % behind the fastest on average, 9 % at worst.
    const int steps = (a.cells / 32 + 7) / 8, share = *lds <= 80 * 1024 ? 2 : 1, rounds = (*grid + share * num_cu - 1) / (share * num_cu);
    const double one = a.chunks * (1.02 + 0.000376 * (c.mf * a.cells + c.mc * a.xcells) + 0.0134 * steps * (2.25 * c.mf * c.mc + 9 * c.mc + c.mf));
    const double t = *grid <= num_cu ? one : rounds * one * (1.0 + 0.21 * (std::min((double)share, *grid / (double)num_cu) - 1.0));
    const double moved = 4.82e-6 * a.chunks * (c.mf * a.cells + c.mc * a.xcells) * *grid;
    *est = 3.1 + cbrt(t * t * t + moved * moved * moved) + rounds * c.mf * c.mc * (copies == 4 ? 0.506 : 0.103);
    *out = a;
    return true;
}

int pc_wgrad_few_tile(const pc_conv_desc *d, int num_cu, double limit)
{
    if (d->stride != 1 || (d->C & 7) || (d->F & 7)) return -1;
    int best = -1;
    for (int k = 0; k < 4; ++k) {
        FewWgradArgs a;
        size_t lds;
        int grid;
        double us;
        if (plan_few(d, kFew[k], num_cu, &a, &lds, &grid, &us) && us < limit) { limit = us; best = k; }
    }
    return best;
}

pc_status pc_mfma_bwd_weight_few(pc_ctx *ctx, const pc_conv_desc *d, const pc_packed *pk, const void *x, const void *dy, float *dw, int tile, bool *launched)
{
    *launched = false;
    FewWgradArgs a;
    size_t lds;
    int grid;
    double us;
    if (d->stride != 1 || (d->C & 7) || (d->F & 7) || !pc_direct_loads(x) || !pc_direct_loads(dy) || !plan_few(d, kFew[tile], ctx->num_cu, &a, &lds, &grid, &us)) return PC_OK;
    static pc_per_device_once attr[4];
    if (pc_once_pending(attr[tile], ctx->device)) {
        PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kFewKernels[tile]), hipFuncAttributeMaxDynamicSharedMemorySize, FW_LDS_MAX));
        pc_once_done(attr[tile], ctx->device);
    }
    hipLaunchKernelGGL(kFewKernels[tile], dim3((unsigned)grid), dim3(512), lds, ctx->stream, (const uint16_t *)x, (const uint16_t *)dy, a, pk->v.kinfo, (float4 *)dw);
    *launched = true;
    pc_note_kernel(ctx, "pc_mfma_wgrad_dma_few_kernel<%d, %d>", kFew[tile].mf, kFew[tile].mc);
    return pc_hip_check(ctx, hipGetLastError(), "MFMA bwd_weight (few pixels) launch");
}
