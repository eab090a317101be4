// Float32 layers on the matrix cores (Section 5.2, forward and backward phase). Tiles of 32 of the forward and backward-data passes
// and the weight gradients: bfloat16 instructions over operands split in three; tiles of 16 and the first layer's weight gradients:
// v_mfma_f32_16x16x4_f32 / 32x32x2_f32.
//
// Three parts. A float32 value is the sum of three bfloat16 values (8 significant bits each, round to nearest, the remainder
// goes on; |a1| <= 2^-8 |a0|, |a2| <= 2^-17 |a0|), and of the nine products of two such sums the six of 2^-16 and above are formed: a
// product of two bfloat16 values is exact in float32, what is left out is at most 2^-24 of a product and 2^-27.5 in the mean square. a0 b0 is
// summed in one accumulator, the five small ones in another, and the two are added once at the end. Error against 64 bits, root mean square relative to the
// result's (normal data; 89 % zero weights in brackets): 64 products 1.43e-7 with v_mfma_f32_32x32x2_f32, 0.50e-7 in parts (0.57,
// 0.29); 1152 products 5.99e-7, 2.00e-7 (2.16, 0.81); 4608 products 11.9e-7, 4.2e-7 (4.2, 1.7): the float32 instruction rounds its sum
// after every two products, this one after sixteen. (All six in one accumulator: 5.2e-7 for 1152, 3.9e-7 with zeros, so two.)
// Small operands: bfloat16 has float32's exponents but ends at 2^-133, so the last parts of an operand under 2^-109 would vanish. Every operand is
// split times 2^16, which puts the last bit of a subnormal, 2^-149, at 2^-133 (the instruction takes subnormal operands), and the sums are
// multiplied by 2^-32 at the end. (64 x 28 x 28, 128 -> 128 forward and backward-data 67.3 -> 70.8 us, 9 x 73 x 74, 416 -> 16 backward-data
// 56.7 -> 61.6, weight gradients up to 2 %.) Operands of 2^112 and sums of 2^96 and above overflow then.
// What does not come out finite, infinities and NaN among the operands too, goes to pc_f32_kept_taps.
// Six products take 192 cycles where the float32 instruction takes 512 for the same tile and depth. 64 x 28 x 28, 128 -> 128:
// forward 132.5 -> 65.6 us, backward-data 133.2 -> 67.3 us (1.3 PFLOP/s of bfloat16 products), 69.0 and 71.9 with the scaling. A wavefront that split its weights itself
// spent 52 vector instructions per 12 matrix instructions on it, and matrix and vector instructions hardly overlap here (busy 58 and 54 % of the
// time, sum 1.12): layers of up to PC_F32_PARTS kernels have their weights split when they are packed, 61.6 and 64.9 us (matrix cores busy 69 %;
// 7.5 -> 3.0 vector instructions per matrix instruction; 16 x 14 x 14, 256 -> 256 31 -> 24 us). Bound now by the barriers of the staging with two
// workgroups per CU and by the split of the pixels. (Tiles of 16 over split weights, with 16x16x32_bf16: 0.6 % on 215 layers, not kept.)
//
// The gather kernels of pc_conv_valu.hip multiply kept taps only, but every multiply-add takes an LDS word and every kept
// kernel a chain of scalar loads: they reach 2 % of the vector rate. The zero-filled contraction runs at the matrix rate whatever the density.
//
// Operand layout: of 32x32x2_f32, lane l holds row (A) / column (B) l % 32 and k = l / 32; of 32x32x16_bf16, the same row and k = 8 (l / 32)
// .. + 7; accumulator register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l % 32. The packed float32 operand holds fragments of 8
// reduction entries: 64 pieces of 16 bytes, piece l the entries 4 (l / 32) .. + 3 of row l % 32; the one in three parts fragments of 16: per
// part 64 pieces of 16 bytes, piece l the lane's eight entries.
//
// The float32 matrix instructions occupy the vector units: a vector instruction of any wavefront of the SIMD adds its four
// cycles to the kernel's time (measured: taking out the loads, the LDS writes and the LDS reads of the weight-gradient loop
// one after the other gives back 9, 8 and 10 %, exactly their vector instructions). So the loops keep addresses in scalar
// offsets of buffer loads and in immediate offsets of LDS reads, let the range check of a buffer load supply the zeros of
// the padding, and copy no operand registers.
#include "pc_mfma.h"
#include <math.h>
#include <algorithm>
#include <type_traits>

// ------------------------------------------------------------------ forward / backward-data
// A workgroup computes 32*WM output channels x 32*WN pixels, one 32 x 32 tile per wavefront (WK = 4: one tile, the four
// wavefronts split the reduction and add up in wavefront order). The pixels of a tile are consecutive in raster order
// over (image, row, column of a strip of Ws columns), so a tile is full whatever the map size; what it reads is a
// range of rows of the "virtual" image in which the images follow each other with one zero row between them. (NT = 2: a wavefront has
// two tiles of pixels and splits its weights once for both.) Staged pixels of tiles of 32: per 16 channels the three parts, 32 bytes each.
// Several workgroups share a CU: the staging of one runs under the matrix instructions of the others.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
// 16-byte elements staged per thread and chunk, tiles of T = 32 or 16
__host__ __device__ constexpr int f32_ne(int T, int NT) { return T == 32 && NT == 1 ? 6 : 8; }

struct F32Class {
    int32_t GH, GW, ooff_y, ooff_x;   // pixel grid of this launch part; output pixel = grid * oscale + ooff
    int32_t Ws, tiles;                // strip width, tiles per strip
    int32_t R, IW;                    // staged rows and columns
    int32_t first;                    // first workgroup of this part
    int32_t ntaps;
    int32_t o0, dr, ds;               // the full 3 x 3: tap 3r + s at LDS byte offset o0 + r*dr + s*ds
    int32_t tap_w[4], tap_off[4];     // a part with fewer taps: weight tap and LDS byte offset
};

struct F32ConvArgs {
    int32_t N, in_H, in_W, in_CH, out_H, out_W, out_CH;
    int32_t oscale, lstep, HP, ioff;  // virtual row v is input row v % HP + ioff (HP = in_H + 1)
    int32_t KC, lparts, nchunk, KS;   // channels per chunk (16 to 128), log2(KC / 4), chunks, fragments of 8 per tap in the operand
    int32_t pitch;                    // bytes per staged pixel
    int32_t m_tiles, ncls;
    int32_t tail_first, tail_R;       // tiles and workgroups from tail_first on: a workgroup per part of 32 x 32; its staged rows
    int32_t act;
    int32_t back, k_row, k_red;       // backward-data; strides of kinfo over output and reduction channels
    const float *act_mask;
    const uint32_t *kinfo;            // pattern masks of the kernels
    F32Class cls[4];
    const uint16_t *w3;               // the weights in three parts, or none
};

// Output channel m of output pixel (oy, ox) of image n, over kept taps inside the map only. The matrix instructions multiply the
// pruned taps of the zero-filled operand too, and 0 x Inf = 0 x NaN = NaN: an element that did not come out finite is computed
// again here, so that what lies under a pruned tap never reaches it.
// (So does the split of an infinity, a NaN or a value that rounds up to a bfloat16 infinity: Inf - Inf and Inf x 0 in the small parts are
// NaN.) (The check of finite tiles is 16 multiply-adds per lane: 28 x 28, 128 -> 128, batch 64 takes 70.2 us without and 70.8 with it.)
__device__ __forceinline__ float pc_f32_kept_taps(const float *__restrict__ in, const float *__restrict__ wz, const F32ConvArgs &g, int n, int oy, int ox, int m)
{
    const float *img = in + (int64_t)n * g.in_H * g.in_W * g.in_CH, *wrow = wz + (int64_t)(m >> 5) * 9 * g.KS * 256 + (m & 31) * 4;
    float acc = 0.0f;
    for (int k0 = 0; k0 < g.in_CH && acc == acc; k0 += 4) {
        uint32_t info[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) info[i] = g.kinfo[m * g.k_row + (k0 + i < g.in_CH ? k0 + i : k0) * g.k_red];
        for (int i = 0; i < 4 && k0 + i < g.in_CH; ++i) {
            const uint32_t u = i == 0 ? info[0] : i == 1 ? info[1] : i == 2 ? info[2] : info[3];
            if (u == 0xFFFFFFFFu) continue;
            const int k = k0 + i;
            const float *wk = wrow + (k >> 3) * 256 + (k >> 2 & 1) * 128 + (k & 3);
            uint32_t left = u & 511u;
            float x[4], w[4];
            bool on[4];
#pragma unroll
            for (int j = 0; j < 4; ++j, left &= left - 1u) {
                const int t = __ffs((int)left) - 1, r = t / 3, s = t - 3 * r;
                int iy = oy * g.lstep + r - 1, ix = ox * g.lstep + s - 1;
                bool hit = true;
                if (g.back) {
                    iy = oy + 1 - r;
                    ix = ox + 1 - s;
                    hit = ((iy | ix) & (g.oscale - 1)) == 0;
                    iy >>= g.oscale - 1;
                    ix >>= g.oscale - 1;
                }
                on[j] = hit && (unsigned)iy < (unsigned)g.in_H && (unsigned)ix < (unsigned)g.in_W;
                x[j] = img[on[j] ? ((int64_t)iy * g.in_W + ix) * g.in_CH + k : 0];
                w[j] = wk[(int64_t)t * g.KS * 256];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = on[j] ? fmaf(x[j], w[j], acc) : acc;
        }
    }
    return acc;
}

template <int T, int NTAPS, int WM, int WN, int WK, int NT, bool VEC, bool PARTS>
__device__ __forceinline__ void pc_f32_conv_body(const float *__restrict__ in, float *__restrict__ out, const float *__restrict__ wz,
                                                 const F32ConvArgs &g, const F32Class &c, int rows, int mt, int strip, int p0,
                                                 unsigned char *lds)
{
    constexpr int FR = 16, F32_NE = f32_ne(T, NT);             // FR: channels per fragment
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave % WK, wn = (wave / WK) % WN, wm = wave / WK / WN;
    const int x0 = strip * c.Ws;
    const int np = g.N * c.GH * c.Ws;
    const int r0 = p0 / c.Ws, n0 = r0 / c.GH, v0 = n0 * g.HP + (r0 - n0 * c.GH) * g.lstep;

    // this lane's pixels: image, row and column of the strip (found again at the end: the registers are needed between)
    struct Pixel { int n, y, x; };
    const int pl = p0 + wn * NT * T + (lane & (T - 1));
    auto pixel = [&](int p) -> Pixel {
        const int r = p / c.Ws, n = r / c.GH;
        return Pixel{n, r - n * c.GH, p - r * c.Ws};
    };
    const unsigned char *bp[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const Pixel q = pixel(pl + j * T < np ? pl + j * T : np - 1);
        bp[j] = lds + ((q.n * g.HP + q.y * g.lstep - v0) * c.IW + q.x * g.lstep) * g.pitch + lane / T * 16;
    }

    // elements this thread stages: 16 bytes (4 channels, the same ones of every pixel) of a pixel each; pix = the input
    // pixel counted from the first image of the tile
    const int total = (rows * c.IW) << g.lparts;
    const int part = (int)threadIdx.x & ((1 << g.lparts) - 1), q0 = (int)threadIdx.x >> g.lparts, dq = 256 >> g.lparts;
    const float *in0 = in + (int64_t)n0 * g.in_H * g.in_W * g.in_CH + part * 4;
    uint32_t pix[F32_NE];
#pragma unroll
    for (int i = 0; i < F32_NE; ++i) {
        const int q = q0 + i * dq;
        const int iy = q / c.IW, ix = q - iy * c.IW;
        const int v = v0 + iy, n = v / g.HP, y = v - n * g.HP + g.ioff, x = x0 * g.lstep + ix + g.ioff;
        const bool ok = iy < rows && n < g.N && y >= 0 && y < g.in_H && x >= 0 && x < g.in_W;
        pix[i] = ok ? (uint32_t)(((n - n0) * g.in_H + y) * g.in_W + x) : 0xFFFFFFFFu;
    }
    // VEC: rows of whole quads, and the images a tile touches within 2 GiB: buffer loads, zeros come from the range check.
    // Else element by element through 64-bit addresses. (Loads stand under no condition: one that does merges with the
    // register's old value, and the copy waits for it.)
    constexpr uint32_t OOB = 0x80000000u;
    const __amdgpu_buffer_rsrc_t isrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(in + (int64_t)n0 * g.in_H * g.in_W * g.in_CH), 0, 0x7FFFFFFF, 0x00020000);
    if (VEC) {
#pragma unroll
        for (int i = 0; i < F32_NE; ++i) pix[i] = pix[i] != 0xFFFFFFFFu ? pix[i] * (uint32_t)(g.in_CH * 4) + part * 16 : OOB;
    }
    const bool part_in_last = (g.nchunk - 1) * g.KC + part * 4 < g.in_CH;
    v4u32 R[F32_NE];
    auto issue = [&](int ch) {
        const int c0 = ch * g.KC;
        const bool cut = ch == g.nchunk - 1 && !part_in_last;
#pragma unroll
        for (int i = 0; i < F32_NE; ++i) {
            if (VEC) {
                R[i] = __builtin_amdgcn_raw_buffer_load_b128(isrc, (int)(cut ? OOB : pix[i]), c0 * 4, 0);
            } else {
                float t[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const bool ok = pix[i] != 0xFFFFFFFFu && c0 + part * 4 + k < g.in_CH;
                    t[k] = *(ok ? in0 + ((uint64_t)pix[i] * (uint32_t)g.in_CH + c0 + k) : in);
                }
                __builtin_memcpy(&R[i], t, 16);
            }
        }
    };
    auto put = [&](int ch) {
        unsigned char *dst = lds + q0 * g.pitch + (T == 32 ? (part >> 2) * 96 + (part & 3) * 8 : part * 16);
        const int left = g.in_CH - ch * g.KC - part * 4;
#pragma unroll
        for (int i = 0; i < F32_NE; ++i)
            if ((int)threadIdx.x + 256 * i < total) {
                if (!VEC) {           // (zeros go in here: a select behind the load would wait for it)
                    const bool ok = pix[i] != 0xFFFFFFFFu;
#pragma unroll
                    for (int k = 0; k < 4; ++k) R[i][k] = ok && left > k ? R[i][k] : 0u;
                }
                if (T == 32) {
                    uint32_t s[2][3];
#pragma unroll
                    for (int e = 0; e < 2; ++e) f32_split(__uint_as_float(R[i][2 * e]), __uint_as_float(R[i][2 * e + 1]), s[e]);
#pragma unroll
                    for (int k = 0; k < 3; ++k) *reinterpret_cast<v2u32 *>(dst + i * dq * g.pitch + k * 32) = v2u32{s[0][k], s[1][k]};
                } else {
                    *reinterpret_cast<v4u32 *>(dst + i * dq * g.pitch) = R[i];
                }
            }
    };

    // a row tile past the last reads the last (not stored)
    int rt = mt * WM + wm;
    const int rt_last = (g.out_CH - 1) / T;
    if (rt > rt_last) rt = rt_last;
    const int KSF = (g.KS + 1) >> 1;
    auto tap_off = [&](int tap) -> int { return NTAPS == 9 ? c.o0 + tap / 3 * c.dr + tap % 3 * c.ds : c.tap_off[tap & 3]; };
    issue(0);
    const int KF = g.KC / FR;
    typename std::conditional<T == 32, f32x16, f32x4>::type acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < T * T / 64; ++i) acc[j][i] = 0.0f;
    if constexpr (T == 32) {
        // WK = 4: wavefronts 0, 1 take the even fragments of 16 channels and 2, 3 the odd ones, each the first or the last taps
        constexpr int HT = WK == 4 ? (NTAPS + 1) / 2 : NTAPS, FS = WK == 4 ? 2 : 1;
        constexpr int RB = HT % 3 == 0 ? 3 : HT % 2 == 0 ? 2 : HT, PD = HT == 9 ? 3 : HT;   // rings of operands and of weights on their way
        const int wf = WK == 4 ? wk >> 1 : 0, t0 = WK == 4 ? (wk & 1) * HT : 0, nt = WK == 4 ? (wk & 1 ? NTAPS - HT : HT) : HT;
        f32x16 low[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) low[j][i] = 0.0f;
        const auto tap = [&](int i) -> int { return WK == 4 ? (t0 + i < NTAPS ? t0 + i : NTAPS - 1) : i; };
        int to[HT];
#pragma unroll
        for (int i = 0; i < HT; ++i) to[i] = tap_off(tap(i));
        // PARTS: weights split at pack time. HT >= 4: a tap's registers are loaded again as soon as its matrix instructions have read them;
        // fewer taps come through registers of their own, for the lead of a whole tap. Else: weights split here, the registers of
        // a tap are free once its parts are made.
        const __amdgpu_buffer_rsrc_t wsrc = PARTS ?
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(g.w3 + (int64_t)rt * 9 * KSF * 1536), 0, 9 * KSF * 3072, 0x00020000) :
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(wz + (int64_t)rt * 9 * KSF * 512), 0, 9 * KSF * 2048, 0x00020000);
        struct Whole { float4 h[2]; };
        typedef typename std::conditional<PARTS, F32Parts, Whole>::type Weights;
        auto a_load = [&](int tap, int kf) -> Weights {
            constexpr int NB = (int)sizeof(Weights) / 16;
            const int tw = NTAPS == 9 ? tap : c.tap_w[tap & 3], at = (tw * KSF + (kf < KSF ? kf : KSF - 1)) * NB * 1024;
            v4u32 u[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k)
                u[k] = __builtin_amdgcn_raw_buffer_load_b128(wsrc, PARTS ? lane * 16 + k * 1024 : (lane >> 5) * 1024 + (lane & 31) * 16 + k * 512, at, 0);
            Weights r;
            __builtin_memcpy(&r, u, sizeof(r));
            return r;
        };
        auto parts = [&](const Weights &w) -> F32Parts {
            if constexpr (PARTS) return w;
            else return f32_split8(w.h[0], w.h[1]);
        };
        constexpr bool IN_PLACE = PARTS && HT >= 4;
        Weights ar[PD];
        F32Parts cur, bq[RB][NT];
#pragma unroll
        for (int i = 0; i < PD; ++i) ar[i] = a_load(tap(i), wf);
        auto b_load = [&](F32Parts *b, int i, int f) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int k = 0; k < 3; ++k) b[j].p[k] = *reinterpret_cast<const bf16x8 *>(bp[j] + f * 96 + to[i] + k * 32);
        };
        if (!IN_PLACE) cur = parts(ar[0]);
        for (int ch = 0; ch < g.nchunk; ++ch) {
            if (ch) __syncthreads();
            __builtin_amdgcn_s_setprio(0);        // a wavefront that multiplies goes first (4 x 71 x 74, 96 -> 96: 25.2 -> 24.6 us)
            put(ch);
            __syncthreads();
            if (ch + 1 < g.nchunk) issue(ch + 1);
            __builtin_amdgcn_s_setprio(1);
            const int left = (g.in_CH - ch * g.KC + FR - 1) / FR, nf = left < KF ? left : KF;
            if (wf >= nf) continue;
            b_load(bq[0], 0, wf);
            for (int f = wf; f < nf; f += FS) {
                const int fn = f + FS < nf ? f + FS : f;
                const int kc = ch * KF + f, kn = f + FS < nf ? ch * KF + fn : (ch + 1) * KF + wf;   // this fragment, the one after it
#pragma unroll
                for (int i = 0; i < HT; ++i) {
                    if (RB > 1) b_load(bq[(i + 1) % RB], i + 1 < HT ? i + 1 : 0, i + 1 < HT ? f : fn);
                    if (!IN_PLACE) ar[i % PD] = a_load(tap((i + PD) % HT), i + PD < HT ? kc : kn);
                    __builtin_amdgcn_sched_barrier(0);
                    if (WK == 1 || i < nt) {
                        const F32Parts *ap = &cur;
                        if constexpr (IN_PLACE) ap = &ar[i % PD];
#pragma unroll
                        for (int m = 0; m < 6; ++m)
#pragma unroll
                            for (int j = 0; j < NT; ++j) {
                                constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
                                f32x16 &s = m == 0 ? acc[j] : low[j];
                                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap->p[PA[m]], bq[i % RB][j].p[PB[m]], s, 0, 0, 0);
                            }
                    }
                    if (!IN_PLACE) cur = parts(ar[(i + 1) % PD]);
                    else ar[i % PD] = a_load(tap((i + PD) % HT), i + PD < HT ? kc : kn);
                    __builtin_amdgcn_sched_barrier(0);
                    if (RB == 1) b_load(bq[0], 0, fn);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[j][i] = WK == 1 ? (acc[j][i] + low[j][i]) * F32_UNSCALE : acc[j][i] + low[j][i];
    } else {
        // One fragment of weights per tap is in flight (a wavefront's loads retire in order: the nine cover the round trip of
        // the next chunk's pixels, which are requested in front of them); LDS reads run one tap ahead. The scheduling barriers
        // keep the loads ahead of the matrix instructions they are to overlap.
        // weights: [row tile of 32][tap][fragment][64 lanes][4]; lane l holds row l % 16 and entries 4 * (l / 16) .. + 3 of 16, two fragments
        // of the 32-row operand; where the second one does not exist its lanes read zeros
        const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(wz + (int64_t)(rt >> 1) * 9 * g.KS * 256), 0, 9 * g.KS * 1024, 0x00020000);
        const uint32_t wvo = (lane >> 5) * 1024u + ((rt & 1) * 16 + (lane & 15) + (lane & 16) * 2) * 16u;
        const uint32_t wvo_last = !(g.KS & 1) || lane < 32 ? wvo : OOB;
        auto a_load = [&](int tap, int kf) -> float4 {
            const int tw = NTAPS == 9 ? tap : c.tap_w[tap & 3];
            const int k = kf < KSF - 1 ? kf : KSF - 1;
            const v4u32 u = __builtin_amdgcn_raw_buffer_load_b128(wsrc, (int)(kf < KSF - 1 ? wvo : wvo_last), (tw * g.KS + k * 2) * 1024, 0);
            float4 r;
            __builtin_memcpy(&r, &u, 16);
            return r;
        };
        auto mma = [&](float a, float bv) { acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bv, acc[0], 0, 0, 0); };
        float4 ar[NTAPS];
#pragma unroll
        for (int t = 0; t < NTAPS; ++t) ar[t] = a_load(t, wk);
        constexpr int RB = NTAPS % 3 == 0 ? 3 : NTAPS % 2 == 0 ? 2 : 1;   // the pixel fragments rotate without copies from one fragment to the next
        float4 bq[RB];
        const unsigned char *bt[NTAPS];
#pragma unroll
        for (int t = 0; t < NTAPS; ++t) bt[t] = bp[0] + tap_off(t);
        for (int ch = 0; ch < g.nchunk; ++ch) {
            if (ch) __syncthreads();
            put(ch);
            __syncthreads();
            if (ch + 1 < g.nchunk) issue(ch + 1);
            const int left = (g.in_CH - ch * g.KC + FR - 1) / FR, nf = left < KF ? left : KF;
            if (wk >= nf) continue;
            bq[0] = *reinterpret_cast<const float4 *>(bt[0] + wk * FR * 4);
            for (int f = wk; f < nf; f += WK) {
                const int fn = f + WK < nf ? f + WK : f;
                const int kn = f + WK < nf ? ch * KF + fn : (ch + 1) * KF + wk;   // the fragment after this one
#pragma unroll
                for (int t = 0; t < NTAPS; ++t) {
                    const float4 a = ar[t], bv = bq[t % RB];
                    if (RB > 1) bq[(t + 1) % RB] = *reinterpret_cast<const float4 *>(t + 1 < NTAPS ? bt[t + 1 < NTAPS ? t + 1 : 0] + f * FR * 4 : bt[0] + fn * FR * 4);
                    __builtin_amdgcn_sched_barrier(0);
                    mma(a.x, bv.x);
                    mma(a.y, bv.y);
                    mma(a.z, bv.z);
                    mma(a.w, bv.w);
                    __builtin_amdgcn_sched_barrier(0);
                    ar[t] = a_load(t, kn);     // behind its last use: the register is free
                    if (RB == 1) bq[0] = *reinterpret_cast<const float4 *>(bt[0] + fn * FR * 4);
                }
            }
        }
    }
    constexpr int NQ = T == 16 || WK > 1 ? 1 : 4;
    float4 o[NT][NQ];
    if constexpr (T == 16) {
        if (WK > 1) {
            // the first wavefront of each pixel tile adds the partial tiles in wavefront order
            float4 *red = reinterpret_cast<float4 *>(lds);
            __syncthreads();
            if (wk) red[(wk * WM * WN + wave / WK) * 64 + lane] = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
            __syncthreads();
            if (wk) return;
#pragma unroll
            for (int k = 1; k < WK; ++k) {
                const float4 u = red[(k * WM * WN + wave / WK) * 64 + lane];
                acc[0][0] += u.x; acc[0][1] += u.y; acc[0][2] += u.z; acc[0][3] += u.w;
            }
        }
        o[0][0] = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
    } else if constexpr (WK > 1) {
        // partial tiles added in wavefront order, wavefront w finishes rows 8w .. 8w+7
        float4 *red = reinterpret_cast<float4 *>(lds);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) red[(wave * 4 + q) * 64 + lane] = make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
        __syncthreads();
        float4 s = red[wk * 64 + lane];
#pragma unroll
        for (int k = 1; k < WK; ++k) {
            const float4 u = red[(k * 4 + wk) * 64 + lane];
            s.x += u.x; s.y += u.y; s.z += u.z; s.w += u.w;
        }
        o[0][0] = make_float4(s.x * F32_UNSCALE, s.y * F32_UNSCALE, s.z * F32_UNSCALE, s.w * F32_UNSCALE);
    } else {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) o[j][q] = make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
    }
    const int m0 = (mt * WM + wm) * T + (T == 32 && WK > 1 ? wk : 0) * 8 + lane / T * 4;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        int p = pl + j * T;
        asm volatile("" : "+v"(p));   // (the compiler would keep the pixels of the start)
        if (p >= np) break;
        const Pixel px = pixel(p);
        if (x0 + px.x >= c.GW) continue;
        const int oy = px.y * g.oscale + c.ooff_y, ox = (x0 + px.x) * g.oscale + c.ooff_x;
        const int64_t opix = ((int64_t)px.n * g.out_H + oy) * g.out_W + ox;
        float z = 0.0f;               // NaN when one of the elements is not finite
        uint32_t redo = 0u;
#pragma unroll
        for (int q = 0; q < NQ; ++q) z = fmaf(o[j][q].x, 0.0f, fmaf(o[j][q].y, 0.0f, fmaf(o[j][q].z, 0.0f, fmaf(o[j][q].w, 0.0f, z))));
        if (__builtin_expect(z != z, 0)) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const float v[4] = {o[j][q].x, o[j][q].y, o[j][q].z, o[j][q].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) redo |= fabsf(v[e]) < INFINITY ? 0u : 1u << (4 * q + e);
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int m = m0 + 8 * q;
            if (m >= g.out_CH) continue;
            const int64_t at = opix * g.out_CH + m;
            float v[4] = {o[j][q].x, o[j][q].y, o[j][q].z, o[j][q].w};
            const int ne = (g.out_CH & 3) == 0 ? 4 : (g.out_CH - m < 4 ? g.out_CH - m : 4);
            if (g.act == PC_ACT_RELU) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
            } else if (g.act == PC_ACT_RELU_MASK) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (e < ne && g.act_mask[at + e] > 0.0f) ? v[e] : 0.0f;
            }
            if ((g.out_CH & 3) == 0) *reinterpret_cast<float4 *>(out + at) = make_float4(v[0], v[1], v[2], v[3]);
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < ne) out[at + e] = v[e];
        }
        for (; redo; redo &= redo - 1u) {
            const int i = __ffs((int)redo) - 1, m = m0 + (i >> 2) * 8 + (i & 3);
            if (m >= g.out_CH) continue;
            float v = pc_f32_kept_taps(in, wz, g, px.n, oy, ox, m);
            if (g.act == PC_ACT_RELU || g.act == PC_ACT_RELU_MASK) v = (g.act == PC_ACT_RELU ? v : g.act_mask[opix * g.out_CH + m]) > 0.0f ? v : 0.0f;
            out[opix * g.out_CH + m] = v;
        }
    }
}

// MC: the four parity classes of a stride-2 backward-data pass (4, 2, 2 and 1 taps), each a range of workgroups.
template <int T, int WM, int WN, int WK, int NT, bool MC, bool VEC, bool PARTS>
__global__ void __launch_bounds__(256, T == 16 ? 4 : NT == 1 ? 3 : 2)
pc_f32_conv_kernel(const float *__restrict__ in, float *__restrict__ out, const float *__restrict__ wz, F32ConvArgs g)
{
    extern __shared__ __align__(16) unsigned char lds[];
    int b = (int)blockIdx.x;
    if constexpr (MC) {           // (the parts differ in taps: in launch order they spread over the XCDs)
        int k = 0;
        while (k + 1 < g.ncls && b >= g.cls[k + 1].first) ++k;
        const F32Class &c = g.cls[k];
        b -= c.first;
        const int mt = b % g.m_tiles, pt = b / g.m_tiles, strip = pt / c.tiles, p0 = (pt - strip * c.tiles) * T * WN * NT;
        if (c.ntaps == 4) pc_f32_conv_body<T, 4, WM, WN, WK, NT, VEC, PARTS>(in, out, wz, g, c, c.R, mt, strip, p0, lds);
        else if (c.ntaps == 2) pc_f32_conv_body<T, 2, WM, WN, WK, NT, VEC, PARTS>(in, out, wz, g, c, c.R, mt, strip, p0, lds);
        else pc_f32_conv_body<T, 1, WM, WN, WK, NT, VEC, PARTS>(in, out, wz, g, c, c.R, mt, strip, p0, lds);
    } else {
        const F32Class &c = g.cls[0];
        const bool tail = T == 32 && WK == 1 && b >= g.tail_first;
        int sub = 0;
        if (tail) {
            b -= g.tail_first;
            sub = b % (WM * WN * NT);
            b = g.tail_first + b / (WM * WN * NT);
        } else if ((g.tail_first & 7) == 0) {
            b = (b & 7) * (g.tail_first >> 3) + (b >> 3);   // workgroups that share pixels share an XCD
        }
        const int mt = b % g.m_tiles, pt = b / g.m_tiles, strip = pt / c.tiles, p0 = (pt - strip * c.tiles) * T * WN * NT;
        if constexpr (T == 32 && WK == 1) {
            if (tail) {
                if (p0 + sub / WM * 32 >= g.N * c.GH * c.Ws || (mt * WM + sub % WM) * 32 >= g.out_CH) return;
                pc_f32_conv_body<32, 9, 1, 1, 4, 1, VEC, PARTS>(in, out, wz, g, c, g.tail_R, mt * WM + sub % WM, strip, p0 + sub / WM * 32, lds);
                return;
            }
        }
        pc_f32_conv_body<T, 9, WM, WN, WK, NT, VEC, PARTS>(in, out, wz, g, c, c.R, mt, strip, p0, lds);
    }
}

// ---- plan and launch
// Staged rows of a tile of BN pixels of strips of Ws columns.
static int f32_rows(const F32ConvArgs &g, int GH, int Ws, int ext, int BN)
{
    const int rows = BN % Ws == 0 ? BN / Ws : (BN + Ws - 2) / Ws + 1;         // output rows a tile touches at most
    const int cross = (rows - 1 + GH - 1) / GH;                               // image boundaries among them
    const int gap = g.HP - GH * g.lstep;                                      // virtual rows between two images beyond the step
    return (rows - 1) * g.lstep + cross * (gap > 0 ? gap : 0) + ext;
}

// Strips and staged extent of one part for BN pixels per tile; false when it does not fit the staging registers.
static bool f32_plan_class(const F32ConvArgs &g, F32Class *c, int ext, int BN, int NE)
{
    int64_t best = -1;
    for (int ns = 1, Ws = c->GW; Ws >= 1; ns = Ws > 1 ? (c->GW + Ws - 2) / (Ws - 1) : 1, Ws = Ws > 1 ? (c->GW + ns - 1) / ns : 0) {
        const int64_t np = (int64_t)g.N * c->GH * Ws;
        if (np + BN >= ((int64_t)1 << 31)) continue;
        const int64_t vr = (int64_t)g.N * g.HP + 8;
        if (vr >= ((int64_t)1 << 31)) return false;
        const int R = f32_rows(g, c->GH, Ws, ext, BN), IW = (Ws - 1) * g.lstep + ext;
        if ((int64_t)R * IW * (g.KC / 4) > 256 * NE) continue;
        // columns past the map cost matrix work, staged pixels cost less
        const int64_t cost = (int64_t)ns * Ws * (8 * BN + R * IW);
        if (best < 0 || cost < best) {
            best = cost;
            c->Ws = Ws; c->R = R; c->IW = IW;
            c->tiles = (int)((np + BN - 1) / BN);
        }
    }
    return best >= 0;
}

// Tile shapes: a workgroup's tile is T*wm output channels x T*wn pixels, wk wavefronts split its reduction; `mma` is the time of
// its matrix instructions in units of their issue cycles. Tiles of 16 x 16 have a quarter of the work per workgroup: layers
// with few pixels fill the chip (2 x 11 x 13, 360 -> 24 forward: 9 tiles of 32 took 21.9 us, 42 of 16 take 9.3), and
// layers of up to 16 output channels do half the matrix work (45 x 44, 384 -> 16: 21.7 -> 9.2 us). The larger tiles read
// fewer weights and pixels per multiply-add and win where there are enough of them.
// Tiles of 32: nt = 2 pixel tiles per wavefront halve the splitting of the weights and their loads and win where two workgroups per CU
// are enough of them (64 x 28 x 28, 128 -> 128 forward 75.4 -> 65.7 us), nt = 1 has three per CU.
struct F32Shape { int t, wm, wn, wk, nt; double mma, mma_parts; };   // mma_parts: over weights split at pack time
static const F32Shape kF32Shapes[] = {{32, 2, 2, 1, 2, 0.803, 0.762}, {32, 4, 1, 1, 2, 0.781, 0.695}, {32, 1, 4, 1, 2, 0.836, 0.698},
                                      {32, 2, 2, 1, 1, 0.901, 0.683}, {32, 4, 1, 1, 1, 0.856, 0.586}, {32, 1, 4, 1, 1, 0.937, 0.656},
                                      {32, 1, 1, 4, 1, 1.066, 0.922},
                                      {16, 1, 4, 1, 1, 0.733, 0.0}, {16, 1, 2, 2, 1, 0.658, 0.0}, {16, 1, 1, 4, 1, 0.567, 0.0}};
// The rest of the estimate, by kind: tiles of 16; of 32 with one and with two pixel tiles per wavefront; of 32 along the reduction; and
// those of 32 again over weights split at pack time
struct F32Kind { int occ; double alone, part_round, stage, start, trip; };
static const F32Kind kF32Kinds[] = {{4, 0.495, 0.962, 141.0, 1243.0, 740.0}, {3, 0.469, 0.613, 218.0, 1777.0, 1247.0},
                                    {2, 0.928, 0.816, 218.0, 1777.0, 1247.0}, {3, 0.469, 0.476, 218.0, 1777.0, 1247.0},
                                    {3, 0.318, 0.669, 223.0, 1866.0, 1290.0}, {2, 0.347, 0.730, 247.0, 2466.0, 1788.0},
                                    {3, 1.361, 0.771, 190.0, 1437.0, 739.0}};
static const F32Kind &f32_kind(const F32Shape &s, bool parts) { return kF32Kinds[s.t == 16 ? 0 : (s.wk > 1 ? 3 : s.nt) + (parts ? 3 : 0)]; }

// Time estimate in us, least squares over 14000 measured launches (400 layers of 1 .. 128 images, 4 .. 224 pixels wide, 1 .. 512 channels,
// both passes and strides; the choice was 1.3 % behind the best shape on average, 2.7 % in backward-data passes of stride 2, the worst
// one 31 %), and for weights split at pack time over 7500 more (494 layers and passes: 1.5 % forward, 1.3 % backward-data, 1.8 and 3.8 % at stride 2,
// the worst 25 %; with the figures of weights split in the kernel 2.8, 2.6, 1.8, 5.0 and 34 %. profiles/plan_timings_f32.csv has 82 of the
// layers): a workgroup costs its
// matrix cycles (more per cycle the fewer workgroups share the CU), its start and end, staging per 256 elements of 16 bytes, and per
// chunk a round trip that the other workgroups of the CU hide; then the output and the weights from the L2s.
static int f32_occ(const F32Shape &s, size_t lds)
{
    const int occ = (int)(160 * 1024 / lds), most = f32_kind(s, false).occ;
    return occ < most ? occ : most;
}

// Cycles of one workgroup; rounds = workgroups per CU.
static double f32_cycles(const F32Shape &s, const F32ConvArgs &t, double taps, double staged, double rounds, size_t lds)
{
    const F32Kind &q = f32_kind(s, t.w3);
    const int left = t.in_CH - (t.nchunk - 1) * t.KC, wf = s.t == 32 && s.wk == 4 ? 2 : s.wk;
    const int frags = (t.nchunk - 1) * (t.KC / 16 / wf) + ((left + 15) / 16 + wf - 1) / wf;
    if (s.t == 32 && s.wk == 4) taps = (taps + 1.0) / 2.0;
    const double up = ceil(rounds), occ = f32_occ(s, lds), conc = up < occ ? up : occ;
    return taps * frags * (s.t == 16 ? 128.0 * s.mma : 192.0 * s.nt * (t.w3 ? s.mma_parts : s.mma)) * (1.0 + q.alone / conc) + staged / 256.0 * t.nchunk * q.stage + q.start +
           q.trip * t.nchunk / conc;
}

static double f32_rounds(const F32Shape &s, bool parts, double n) { return n <= f32_kind(s, parts).occ ? ceil(n) : n + f32_kind(s, parts).part_round; }

static double f32_time(const pc_ctx *ctx, const F32Shape &s, const F32ConvArgs &t, int64_t blocks, double taps, double staged, size_t lds, int64_t out_bytes)
{
    const double n = (double)blocks / ctx->num_cu;
    const double wbytes = (double)blocks * s.t * s.wm * taps * ((t.in_CH + 7) / 8 * 32) * (s.t == 32 && t.w3 ? 1.5 : 1.0);
    return 3.6 + f32_rounds(s, t.w3, n) * f32_cycles(s, t, taps, staged, n, lds) / 2350.0 + (double)out_bytes / 5.5e6 + wbytes / 90e6;
}

// The last, partly filled round of a launch: its tiles are cut into parts of 32 x 32, one workgroup each, four wavefronts along the
// reduction. What bounds such a launch is the time of whole tiles on the CUs that have one more than the others; a part takes
// a quarter of a tile's time or less, so the CUs end that much closer together. Taken where the estimate is at least 2 % shorter
// (parts stage and read more per multiply-add, and LDS for their sums may cost a workgroup per CU). 34 layers, with float32 instructions, in us: 64 x 28 x 28,
// 128 -> 128 forward 128.9 -> 119.7 (6.1 tiles per CU), backward-data 125.1 -> 111.8; 117 x 119, 72 -> 136 68.8 -> 53.1;
// geometric mean 1.08 and 1.06, the least 0.96. Tiles of 16 end in small steps by themselves, and launches of the parity classes of
// stride 2 mix short and long workgroups, so neither is cut.
static void f32_plan_tail(const pc_ctx *ctx, const F32Shape &s, F32ConvArgs *t, int ext, int64_t *blocks, double staged, size_t *lds, double *us)
{
    static const F32Shape part = {32, 1, 1, 4, 1, 1.066, 0.922};
    const F32Class &c = t->cls[0];
    const int sub = s.wm * s.wn * s.nt;
    const int64_t whole = *blocks / ctx->num_cu * ctx->num_cu, rest = *blocks - whole;
    const int R = f32_rows(*t, c.GH, c.Ws, ext, 32);
    if (whole == 0 || rest == 0 || R * c.IW * 8 > 256 * f32_ne(32, 1) || R > c.R || whole + rest * sub >= ((int64_t)1 << 31)) return;
    const size_t need = *lds < 16384 ? 16384 : *lds;   // (the parts add their four sums there)
    const double n = (double)*blocks / ctx->num_cu, k = (double)(whole / ctx->num_cu), m = (double)(rest * sub) / ctx->num_cu;
    const double now = f32_rounds(s, t->w3, n) * f32_cycles(s, *t, 9.0, staged, n, *lds);
    const double cut = k * f32_cycles(s, *t, 9.0, staged, n, need) + f32_rounds(part, t->w3, m) * f32_cycles(part, *t, 9.0, (double)R * c.IW * 8, n, need);
    if (cut >= 0.98 * now) return;
    *us -= (now - cut) / 2350.0;
    t->tail_first = (int32_t)whole;
    t->tail_R = R;
    *blocks = whole + rest * sub;
    *lds = need;
}

// g holds the tensors' extents; cls[].{GH, GW, ooff, ntaps, tap_w} and the tap positions tr, tc are set.
static pc_status f32_run(pc_ctx *ctx, F32ConvArgs g, bool mc, int ext, const int (*tr)[9], const int (*tc)[9], const float *in, float *out,
                         const float *wz)
{
    F32ConvArgs best;
    int best_k = -1;
    int64_t best_blocks = 0;
    size_t lds = 0;
    double best_us = 0.0;
    const int c8 = (g.in_CH + 7) / 8 * 8;
    const int64_t out_bytes = (int64_t)g.N * g.out_H * g.out_W * g.out_CH * 4;
    const int32_t key[PC_CHOICE_KEY] = {1, g.N, g.in_H, g.in_W, g.in_CH, g.out_H, g.out_W, g.out_CH, g.lstep, mc};
    bool known;
    int32_t *choice = pc_choice(ctx, key, &known);
    for (int k = 0; k < (int)(sizeof(kF32Shapes) / sizeof(kF32Shapes[0])); ++k) {
        const F32Shape &s = kF32Shapes[k];
        // chunks of 32 (128) channels, shorter ones where the staged tile would not fit, down to one fragment per wavefront
        const int kc_min = 16 * (s.t == 32 && s.wk == 4 ? 2 : s.wk);
        for (int kc = s.t == 16 ? 128 : 32; kc >= kc_min; kc >>= 1) {
            if (known ? *choice != k * 256 + kc : kc >= 2 * c8 && kc > kc_min) continue;
            F32ConvArgs t = g;
            t.KC = kc;
            t.lparts = 0;
            while ((4 << t.lparts) < kc) ++t.lparts;
            t.pitch = t.KC * (s.t == 32 ? 6 : 4) + 16;
            t.nchunk = (g.in_CH + t.KC - 1) / t.KC;
            t.m_tiles = (g.out_CH + s.t * s.wm - 1) / (s.t * s.wm);
            int64_t blocks = 0;
            bool ok = true;
            double taps = 0.0, staged = 0.0;                              // sums over the workgroups
            size_t need = s.wk > 1 ? 16384 : 0;
            for (int i = 0; i < g.ncls && ok; ++i) {
                F32Class &c = t.cls[i];
                ok = f32_plan_class(t, &c, ext, s.t * s.wn * s.nt, f32_ne(s.t, s.nt));
                if (!ok) break;
                const int64_t nb = (int64_t)c.tiles * ((c.GW + c.Ws - 1) / c.Ws) * t.m_tiles;
                c.first = (int32_t)blocks;
                blocks += nb;
                if (blocks >= ((int64_t)1 << 31)) ok = false;
                taps += (double)nb * c.ntaps;
                staged += (double)nb * c.R * c.IW * (kc / 4);
                if ((size_t)c.R * c.IW * t.pitch > need) need = (size_t)c.R * c.IW * t.pitch;
                if (mc) {
                    for (int q = 0; q < c.ntaps; ++q) c.tap_off[q] = (tr[i][q] * c.IW + tc[i][q]) * t.pitch;
                } else {                  // tap rows and columns ascend (forward) or descend (rotated)
                    c.o0 = (tr[i][0] * c.IW + tc[i][0]) * t.pitch;
                    c.dr = (tr[i][3] - tr[i][0]) * c.IW * t.pitch;
                    c.ds = (tc[i][1] - tc[i][0]) * t.pitch;
                }
            }
            if (!ok) continue;
            double us = f32_time(ctx, s, t, blocks, taps / (double)blocks, staged / (double)blocks, need, out_bytes);
            t.tail_first = (int32_t)blocks;
            if (!mc && s.t == 32 && s.wk == 1 && kc == 32) f32_plan_tail(ctx, s, &t, ext, &blocks, staged / (double)blocks, &need, &us);
            if (best_k < 0 || us < best_us) { best = t; best_k = k; best_blocks = blocks; best_us = us; lds = need; }
        }
    }
    if (best_k < 0) return pc_fail(ctx, PC_ERR_UNSUPPORTED, "float32 conv: no tile fits");
    *choice = best_k * 256 + best.KC;
    const dim3 grid((unsigned)best_blocks), blk(256);
    // images a tile may touch: its first one and those the rows of a tile reach into
    int64_t span = 0;
    for (int i = 0; i < best.ncls; ++i) {
        const F32Class &c = best.cls[i];
        const int64_t n = 2 + (kF32Shapes[best_k].t * kF32Shapes[best_k].wn * kF32Shapes[best_k].nt + c.Ws - 1) / c.Ws / c.GH;
        if (n > span) span = n;
    }
    const bool vec = (g.in_CH & 3) == 0 && span * g.in_H * g.in_W * g.in_CH * 4 < ((int64_t)1 << 31);
    hipStream_t st = ctx->stream;
    const bool parts = best.w3 != nullptr && kF32Shapes[best_k].t == 32;
#define F32_LAUNCH_(T, WM, WN, WK, NT, PARTS)                                                                                \
    do {                                                                                                                    \
        if (mc && vec) hipLaunchKernelGGL((pc_f32_conv_kernel<T, WM, WN, WK, NT, true, true, PARTS>), grid, blk, lds, st, in, out, wz, best);   \
        else if (mc) hipLaunchKernelGGL((pc_f32_conv_kernel<T, WM, WN, WK, NT, true, false, PARTS>), grid, blk, lds, st, in, out, wz, best);    \
        else if (vec) hipLaunchKernelGGL((pc_f32_conv_kernel<T, WM, WN, WK, NT, false, true, PARTS>), grid, blk, lds, st, in, out, wz, best);   \
        else hipLaunchKernelGGL((pc_f32_conv_kernel<T, WM, WN, WK, NT, false, false, PARTS>), grid, blk, lds, st, in, out, wz, best);           \
    } while (0)
#define F32_LAUNCH(T, WM, WN, WK, NT)                                                                                        \
    do {                                                                                                                    \
        if (T == 32 && parts) F32_LAUNCH_(T, WM, WN, WK, NT, (T == 32));                                                    \
        else F32_LAUNCH_(T, WM, WN, WK, NT, false);                                                                         \
    } while (0)
    switch (best_k) {
    case 0: F32_LAUNCH(32, 2, 2, 1, 2); break;
    case 1: F32_LAUNCH(32, 4, 1, 1, 2); break;
    case 2: F32_LAUNCH(32, 1, 4, 1, 2); break;
    case 3: F32_LAUNCH(32, 2, 2, 1, 1); break;
    case 4: F32_LAUNCH(32, 4, 1, 1, 1); break;
    case 5: F32_LAUNCH(32, 1, 4, 1, 1); break;
    case 6: F32_LAUNCH(32, 1, 1, 4, 1); break;
    case 7: F32_LAUNCH(16, 1, 4, 1, 1); break;
    case 8: F32_LAUNCH(16, 1, 2, 2, 1); break;
    default: F32_LAUNCH(16, 1, 1, 4, 1); break;
    }
#undef F32_LAUNCH
#undef F32_LAUNCH_
    const F32Shape &bs = kF32Shapes[best_k];
    pc_note_kernel(ctx, "pc_f32_conv_kernel<%d, %d, %d, %d, %d, %s, %s, %s>", bs.t, bs.wm, bs.wn, bs.wk, bs.nt, mc ? "true" : "false", vec ? "true" : "false",
                   parts ? "true" : "false");
    return pc_hip_check(ctx, hipGetLastError(), "float32 conv launch");
}

pc_status pc_f32_fwd(pc_ctx *ctx, const pc_conv_desc *d, const pc_packed *pk, const void *x, void *y, int act)
{
    F32ConvArgs g;
    memset(&g, 0, sizeof(g));
    g.N = d->N; g.in_H = d->H; g.in_W = d->W; g.in_CH = d->C;
    g.out_H = (d->H - 1) / d->stride + 1; g.out_W = (d->W - 1) / d->stride + 1; g.out_CH = d->F;
    g.oscale = 1; g.lstep = d->stride; g.HP = d->H + 1; g.ioff = -1;
    g.KS = pk->v.Ck / 8;
    g.kinfo = pk->v.kinfo; g.k_row = d->C; g.k_red = 1; g.w3 = pk->v.w3_fwd;
    g.act = act; g.ncls = 1;
    F32Class &c = g.cls[0];
    c.GH = g.out_H; c.GW = g.out_W; c.ntaps = 9;
    int tr[1][9], tc[1][9];
    for (int t = 0; t < 9; ++t) { tr[0][t] = t / 3; tc[0][t] = t % 3; }
    return f32_run(ctx, g, false, 3, tr, tc, (const float *)x, (float *)y, (const float *)pk->v.wz_fwd);
}

pc_status pc_f32_bwd_data(pc_ctx *ctx, const pc_conv_desc *d, const pc_packed *pk, const void *dy, void *dx, int act, const void *act_mask)
{
    F32ConvArgs g;
    memset(&g, 0, sizeof(g));
    g.N = d->N; g.in_H = (d->H - 1) / d->stride + 1; g.in_W = (d->W - 1) / d->stride + 1; g.in_CH = d->F;
    g.out_H = d->H; g.out_W = d->W; g.out_CH = d->C;
    g.oscale = d->stride; g.lstep = 1; g.HP = g.in_H + 1;
    g.KS = pk->v.Fk / 8;
    g.back = 1; g.kinfo = pk->v.kinfo; g.k_row = 1; g.k_red = d->C; g.w3 = pk->v.w3_bwd;
    g.act = act; g.act_mask = (const float *)act_mask;
    int tr[4][9], tc[4][9];
    if (d->stride == 1) {
        // dx[iy,ix] reads dy[iy+1-r, ix+1-s]: tap (r,s) at staged offset (2-r, 2-s) from (iy-1, ix-1)
        g.ioff = -1; g.ncls = 1;
        F32Class &c = g.cls[0];
        c.GH = d->H; c.GW = d->W; c.ntaps = 9;
        for (int t = 0; t < 9; ++t) { tr[0][t] = 2 - t / 3; tc[0][t] = 2 - t % 3; }
        return f32_run(ctx, g, false, 3, tr, tc, (const float *)dy, (float *)dx, (const float *)pk->v.wz_bwd);
    }
    // stride 2: input pixel (2a+py, 2b+px) receives tap (r,s) iff py+1-r and px+1-s are even, from dy[a+(py+1-r)/2, b+(px+1-s)/2]
    static const int order[4][2] = {{1, 1}, {1, 0}, {0, 1}, {0, 0}};
    for (int k = 0; k < 4; ++k) {
        const int py = order[k][0], px = order[k][1];
        F32Class &c = g.cls[g.ncls];
        c.GH = (d->H - py + 1) / 2; c.GW = (d->W - px + 1) / 2;
        if (c.GH < 1 || c.GW < 1) continue;
        c.ooff_y = py; c.ooff_x = px;
        for (int t = 0; t < 9; ++t) {
            const int r = t / 3, s = t % 3;
            if ((py + 1 - r) % 2 || (px + 1 - s) % 2) continue;
            c.tap_w[c.ntaps] = t;
            tr[g.ncls][c.ntaps] = (py + 1 - r) / 2; tc[g.ncls][c.ntaps] = (px + 1 - s) / 2;
            ++c.ntaps;
        }
        ++g.ncls;
    }
    return f32_run(ctx, g, true, 2, tr, tc, (const float *)dy, (float *)dx, (const float *)pk->v.wz_bwd);
}

// ------------------------------------------------------------------ backward-weight
// dW[t][f][c] = sum over output pixels of dy[pixel][f] * x[pixel shifted by tap t][c]. The pixels are the reduction. Both sides are split
// in three parts (see above) when they are staged, 4 channels of a pixel at a time, and gfx950's transposing LDS reads make operands of 8
// pixels of one channel per lane from the pixel rows, so a tap is an offset. A wavefront holds 32 filters x 16 channels of all 9 taps (72
// sums, v_mfma_f32_16x16x32_bf16) and multiplies 32 pixels at a time: 66 reads of 8 bytes per 108 matrix instructions of 16 cycles, of the
// LDS's bandwidth 60 %. The small products of 32 pixels start from zero and are added to the sums once: an accumulator of their own for
// every tap does not fit, and in one accumulator with the leading product the error is larger than that of float32 instructions.
// WF x WC wavefronts cover 32*WF filters x 16*WC channels; of fewer than four, the WK = 4 / (WF*WC) that are left over take other
// pixels, and their sums are added in LDS (halves of the tile at a time, a wavefront keeps 8 / WK of its kernels). Pixel tiles are
// split over the workgroups (two per CU); every split writes the kept taps in compact slot order, pc_wgrad_reduce adds the planes in a
// fixed order. 64 x 28 x 28, 128 -> 128, with the sum of the planes: 151 -> 80 us (32 x 32 tiles of v_mfma_f32_32x32x2_f32 before); matrix
// cores busy 54 % of the time, the LDS 40 %. A third wavefront per SIMD would need 168 registers, this takes 195.
// THIN (at most 3 channels): the 9 * C (tap, channel) pairs are the columns of one tile of float32 instructions, one instead of 9.
// 16-byte elements of dy and of x staged per thread and pixel tile (three parts: 32 pixels of dy per wavefront that shares them)
__host__ __device__ constexpr int f32w_nd(int wc, bool thin) { return thin || wc == 2 ? 2 : 4; }
__host__ __device__ constexpr int f32w_nx(bool thin) { return thin ? 6 : 4; }

struct F32WgradArgs {
    int32_t N, H, W, C, F, Ho, Wo, stride;
    int32_t TR, TC, TCe, IR, IW;          // pixel tile, its columns rounded up to even, staged extent of x
    int32_t tiles_r, tiles_c, n_tiles, ksplit, ct, ft;
    int32_t nd, nx;                       // elements per tile
    // multiply-high divisions by TCe / 2, TCe and IW; where `exact` also those of the tile's index and the workgroup's
    uint32_t mg_half, mg_TCe, mg_IW, mg_tc, mg_tr, mg_ks, mg_ct;
    int32_t exact;
    int64_t pstride;                      // slots per partial plane
};

// Words per staged pixel of n channels in three parts: rows of 64 bytes of four pixels in a row stand in different banks
__host__ __device__ constexpr int f32w_pitch(int n) { return n == 64 ? 104 : n == 32 ? 56 : 24; }

template <int WF, int WC, bool THIN, bool VEC>
__global__ void __launch_bounds__(256, 2)
pc_f32_wgrad_kernel(const float *__restrict__ x, const float *__restrict__ dy, F32WgradArgs a, const uint32_t *__restrict__ kinfo,
                    float4 *__restrict__ partial)
{
    extern __shared__ __align__(16) float smem[];
    constexpr int WK = 4 / (WF * WC), FD = 32 * WF, CT = THIN ? 32 : 16, CD = THIN ? 4 : CT * WC;   // CT: columns of a wavefront
    constexpr int F32W_ND = f32w_nd(WC, THIN), F32W_NX = f32w_nx(THIN);
    constexpr int PD = THIN ? FD + 4 : f32w_pitch(FD), PX = THIN ? 4 : f32w_pitch(CD);   // words per staged pixel
    constexpr int NT = THIN ? 1 : 9;
    const int lane = threadIdx.x & 63, h = lane / CT, n32 = lane % CT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave % WK, wc = (wave / WK) % WC, wf = wave / WK / WC;
    auto divide = [&](int q, int d, uint32_t mg) { return a.exact ? (int)pc_udiv((uint32_t)q, mg) : q / d; };
    const int b = (int)blockIdx.x, tile = divide(b, a.ksplit, a.mg_ks), split = b - tile * a.ksplit;
    const int tf = divide(tile, a.ct, a.mg_ct), c0 = (tile - tf * a.ct) * CD, f0 = tf * FD;
    float *sd = smem, *sx = smem + (THIN ? a.TR * a.TCe : 256 * F32W_ND / (FD / 4)) * PD;

    // staged elements: a thread takes the same 4 filters (channels) of several positions; position inside the tile (or
    // its x region) and offset inside an image
    const int dp = (int)threadIdx.x % (FD / 4), dq = (int)threadIdx.x / (FD / 4), xp = (int)threadIdx.x % (CD / 4), xq = (int)threadIdx.x / (CD / 4);
    const int dleft = a.F - (f0 + dp * 4), xleft = a.C - (c0 + xp * 4);
    int dpos[F32W_ND], xpos[F32W_NX], doff[F32W_ND], xoff[F32W_NX];
#pragma unroll
    for (int i = 0; i < F32W_ND; ++i) {
        const int q = dq + i * (1024 / FD), r = (int)pc_udiv((uint32_t)q, a.mg_TCe), col = q - r * a.TCe;
        dpos[i] = r < a.TR && col < a.TC && dleft > 0 ? (r << 16) | col : -1;
        doff[i] = (r * a.Wo + col) * a.F + f0 + dp * 4;
    }
#pragma unroll
    for (int i = 0; i < F32W_NX; ++i) {
        const int q = xq + i * (1024 / CD), r = (int)pc_udiv((uint32_t)q, a.mg_IW), col = q - r * a.IW;
        xpos[i] = r < a.IR && xleft > 0 ? (r << 16) | col : -1;
        xoff[i] = (r * a.W + col) * a.C + c0 + xp * 4;
    }
    constexpr uint32_t OOB = 0x80000000u;
    v4u32 RD[F32W_ND], RX[F32W_NX];
    auto load4 = [&](const float *src, int64_t at, bool ok, int left) -> v4u32 {
        float t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = src[ok && k < left ? at + k : 0];
        v4u32 r;
        __builtin_memcpy(&r, t, 16);
        return r;
    };
    // valid elements of the tile in the registers, one bit each (not VEC: zeros go in when the element goes to LDS, a
    // select behind a load would wait for it); VEC: rows of whole quads, an image within 2 GiB
    uint32_t okd = 0, okx = 0;
    auto issue = [&](int kt) {
        const int q = divide(kt, a.tiles_c, a.mg_tc), tc = kt - q * a.tiles_c, n = divide(q, a.tiles_r, a.mg_tr), tr = q - n * a.tiles_r;
        const int oy = tr * a.TR, ox = tc * a.TC, iy = oy * a.stride - 1, ix = ox * a.stride - 1;
        const float *dimg = dy + (int64_t)n * a.Ho * a.Wo * a.F, *ximg = x + (int64_t)n * a.H * a.W * a.C;
        const int db = (oy * a.Wo + ox) * a.F, xb = (iy * a.W + ix) * a.C;
        const __amdgpu_buffer_rsrc_t dsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(dimg), 0, 0x7FFFFFFF, 0x00020000);
        const __amdgpu_buffer_rsrc_t xsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(ximg), 0, 0x7FFFFFFF, 0x00020000);
        okd = okx = 0;
#pragma unroll
        for (int i = 0; i < F32W_ND; ++i) {
            const bool ok = dpos[i] >= 0 && oy + (dpos[i] >> 16) < a.Ho && ox + (dpos[i] & 0xFFFF) < a.Wo;
            if (VEC) RD[i] = __builtin_amdgcn_raw_buffer_load_b128(dsrc, (int)(ok ? (uint32_t)(db + doff[i]) * 4u : OOB), 0, 0);
            else { RD[i] = load4(dimg, (int64_t)db + doff[i], ok, dleft); okd |= ok ? 1u << i : 0u; }
        }
#pragma unroll
        for (int i = 0; i < F32W_NX; ++i) {
            if (256 * i >= a.nx) break;           // (the same for all)
            const int yy = iy + (xpos[i] >> 16), xx = ix + (xpos[i] & 0xFFFF);
            const bool ok = xpos[i] >= 0 && (unsigned)yy < (unsigned)a.H && (unsigned)xx < (unsigned)a.W;
            if (VEC) RX[i] = __builtin_amdgcn_raw_buffer_load_b128(xsrc, (int)(ok ? (uint32_t)(xb + xoff[i]) * 4u : OOB), 0, 0);
            else { RX[i] = load4(ximg, (int64_t)xb + xoff[i], ok, xleft); okx |= ok ? 1u << i : 0u; }
        }
    };
    auto store = [&](float *at, int part, int channels, const v4u32 &v) __attribute__((always_inline)) {   // 4 channels of a pixel
        if (THIN) {
            *reinterpret_cast<v4u32 *>(at + part * 4) = v;
            return;
        }
        uint32_t s[2][3];
        f32_split(__uint_as_float(v[0]), __uint_as_float(v[1]), s[0]);
        f32_split(__uint_as_float(v[2]), __uint_as_float(v[3]), s[1]);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<v2u32 *>(at + k * (channels / 2) + part * 2) = v2u32{s[0][k], s[1][k]};
    };
    auto put = [&]() {
#pragma unroll
        for (int i = 0; i < F32W_ND; ++i)
            if ((int)threadIdx.x + 256 * i < a.nd) {
                if (!VEC)
#pragma unroll
                    for (int k = 0; k < 4; ++k) RD[i][k] = ((okd >> i) & 1u) && dleft > k ? RD[i][k] : 0u;
                store(sd + (dq + i * (1024 / FD)) * PD, dp, FD, RD[i]);
            }
#pragma unroll
        for (int i = 0; i < F32W_NX; ++i)
            if ((int)threadIdx.x + 256 * i < a.nx) {
                if (!VEC)
#pragma unroll
                    for (int k = 0; k < 4; ++k) RX[i][k] = ((okx >> i) & 1u) && xleft > k ? RX[i][k] : 0u;
                store(sx + (xq + i * (1024 / CD)) * PX, xp, CD, RX[i]);
            }
    };

    // sums of a lane: NV filters of each tap
    constexpr int NV = THIN ? 16 : 8;
    f32x4 acc[NT][NV / 4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < NV / 4; ++q) acc[t][q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int half = a.TCe >> 1, steps = THIN ? a.TR * half : (a.TR * a.TC + 31) >> 5;     // pixel pairs, or groups of 32 pixels
    int kt = split;
    if (kt < a.n_tiles) issue(kt);
    // (compact slot, pattern mask) of the NKER kernels that this lane writes at the end: requested under the last tile, in the registers
    // of its staged elements; behind the loop they would cost a memory round trip
    const int e_tap = THIN && n32 < 9 * a.C ? n32 / a.C : 0;
    const int e_c = THIN ? n32 - e_tap * a.C : c0 + wc * CT + n32;
    const bool e_on = THIN ? n32 < 9 * a.C : e_c < a.C;
    constexpr int NKER = NV / WK;                 // kernels of a lane at the end, and the first of them
    const int v0 = WK == 1 ? 0 : WK == 2 ? wk * (NV / 2) : (wk & 1) * (NV / 2) + (wk >> 1) * (NV / 4);
    auto filter = [&](int r) __attribute__((always_inline)) { return f0 + wf * 32 + (THIN ? 8 : 16) * ((v0 + r) >> 2) + 4 * h + ((v0 + r) & 3); };
    auto kernels = [&]() {
#pragma unroll
        for (int r = 0; r < NKER; ++r) RX[r >> 2][r & 3] = kinfo[e_on && filter(r) < a.F ? (int64_t)filter(r) * a.C + e_c : 0];
    };
    if (kt >= a.n_tiles) kernels();
    if constexpr (THIN) {
        f32x16 sum;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[r] = 0.0f;
        const int a_base = h * PD + wf * 32 + n32;
        const int tap = n32 < 9 * a.C ? n32 / a.C : 0, cn = n32 < 9 * a.C ? n32 - tap * a.C : 0;
        const int b_base = (h * a.stride + tap / 3 * a.IW + tap % 3) * PX + cn;
        // operands of two pixel pairs, used in turn
        float fa[2], fb[2];
        auto read = [&](int s, int k) __attribute__((always_inline)) {
            const int y = (int)pc_udiv((uint32_t)s, a.mg_half), xs = (s - y * half) * 2;
            fa[k] = sd[a_base + (y * a.TCe + xs) * PD];
            fb[k] = sx[b_base + (y * a.IW + xs) * a.stride * PX];
        };
        auto multiply = [&](int k) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            sum = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[k], fb[k], sum, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        for (bool first = true; kt < a.n_tiles; kt += a.ksplit, first = false) {
            if (!first) __syncthreads();
            put();
            __syncthreads();
            if (kt + a.ksplit < a.n_tiles) issue(kt + a.ksplit);
            else kernels();
            // operands of a pixel pair are read one pair ahead (past the last pair: this one again, unused, so that the reads
            // stand under no condition and the waits count them)
            if (wk >= steps) continue;
            read(wk, 0);
            int s = wk;
            for (; s + WK < steps; s += 2 * WK) {
                read(s + WK, 1);
                multiply(0);
                read(s + 2 * WK < steps ? s + 2 * WK : s, 0);
                multiply(1);
            }
            if (s < steps) multiply(0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r >> 2][r & 3] = sum[r];
    } else {
        // Transposing reads: 16 lanes take 4 pixels of 16 channels, lane l gets 4 pixels of channel l % 16; two reads make the lane's 8
        // pixels 8 (l / 16) .. + 7 of the wavefront's 32. Pixels past the tile: zeros of dy, x of pixel 0.
        const int chan = (lane & 3) * 8;
        typedef __attribute__((address_space(3))) i16x4 *lds4;
        int pa[2], pb[2];                         // bytes
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = wk * 32 + 8 * h + 4 * j + (n32 >> 2), q = p < a.TR * a.TC ? p : 0, y = (int)pc_udiv((uint32_t)q, a.mg_TCe);
            pa[j] = (p * PD + wf * 16) * 4 + chan;
            pb[j] = (256 * F32W_ND / (FD / 4) * PD + (y * a.IW + q - y * a.TCe) * a.stride * PX + wc * (CT / 2)) * 4 + chan;
        }
        auto parts = [&](int q0, int q1, int channels) __attribute__((always_inline)) -> F32Parts {
            F32Parts o;
            const unsigned char *p0 = reinterpret_cast<const unsigned char *>(smem) + q0, *p1 = reinterpret_cast<const unsigned char *>(smem) + q1;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p0 + k * channels * 2)), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p1 + k * channels * 2));
                const short __attribute__((ext_vector_type(8))) v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                __builtin_memcpy(&o.p[k], &v, 16);
            }
            return o;
        };
        const int row = a.IW * PX * 4;
        for (bool begin = true; kt < a.n_tiles; kt += a.ksplit, begin = false) {
            if (!begin) __syncthreads();
            __builtin_amdgcn_s_setprio(0);        // a wavefront that multiplies goes first (9 x 73 x 74, 416 -> 16: 122.7 -> 110.8 us)
            put();
            __syncthreads();
            if (kt + a.ksplit < a.n_tiles) issue(kt + a.ksplit);
            else kernels();
            __builtin_amdgcn_s_setprio(1);
            if (wk >= steps) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j) asm volatile("" : "+v"(pb[j]));   // (else the addresses of all taps are held in registers)
            F32Parts A[2], Bq[3];
#pragma unroll
            for (int i = 0; i < 2; ++i) A[i] = parts(pa[0] + i * 32, pa[1] + i * 32, FD);
            Bq[0] = parts(pb[0], pb[1], CD);
            // The small products of a tile start from zero and are added to its sums once: they round below the last bit of these.
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if (t + 1 < NT) {
                    const int at = (t + 1) / 3 * row + (t + 1) % 3 * (PX * 4);
                    Bq[(t + 1) % 3] = parts(pb[0] + at, pb[1] + at, CD);
                }
                __builtin_amdgcn_sched_barrier(0);
                f32x4 low[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                for (int m = 0; m < 6; ++m)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        constexpr int PA[6] = {0, 1, 1, 0, 2, 0}, PB[6] = {1, 0, 1, 2, 0, 0};
                        f32x4 &to = m == 5 ? acc[t][i] : low[i];
                        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i].p[PA[m]], Bq[t % 3].p[PB[m]], to, 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 2; ++i) acc[t][i] += low[i];
            }
        }
    }
    // Sums of wavefronts that shared pixels: partners swap halves of their filters (a wavefront keeps one), of four then quarters.
    if constexpr (WK > 1) {
        constexpr int G = NV / 8;
        f32x4 *mine = reinterpret_cast<f32x4 *>(smem) + wave * (G * NT * 64) + lane;
        const f32x4 *theirs = reinterpret_cast<const f32x4 *>(smem) + (wave ^ 1) * (G * NT * 64) + lane;
        const bool high = wk & 1;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < G; ++j) {
                f32x4 give;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float lo = acc[t][j][i], hi = acc[t][G + j][i];
                    give[i] = high ? lo : hi;
                    acc[t][j][i] = high ? hi : lo;
                }
                mine[(t * G + j) * 64] = give;
                __builtin_amdgcn_sched_barrier(0);
            }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < G; ++j) {
                acc[t][j] += theirs[(t * G + j) * 64];
                if (t % 3 == 2) __builtin_amdgcn_sched_barrier(0);
            }
    }
    if constexpr (WK > 2) {
        constexpr int G = NV / 4;                 // values given away
        typedef float give_t __attribute__((ext_vector_type(G)));
        give_t *mine = reinterpret_cast<give_t *>(smem) + wave * (NT * 64) + lane;
        const give_t *theirs = reinterpret_cast<const give_t *>(smem) + (wave ^ 2) * (NT * 64) + lane;
        const bool high = wk >> 1;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            give_t give;
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const float lo = acc[t][i >> 2][i & 3], hi = acc[t][(G + i) >> 2][(G + i) & 3];
                give[i] = high ? lo : hi;
                acc[t][i >> 2][i & 3] = high ? hi : lo;
            }
            mine[t * 64] = give;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const give_t got = theirs[t * 64];
#pragma unroll
            for (int i = 0; i < G; ++i) acc[t][i >> 2][i & 3] += got[i];
        }
    }
    // kept taps in compact order, straight from the accumulators: a lane holds one channel and NKER filters
    float4 *pout = partial + (int64_t)split * a.pstride;
    uint32_t redo = 0u;                           // kernels with a sum that is not finite
#pragma unroll
    for (int r = 0; r < NKER; ++r) {
        const uint32_t info = RX[r >> 2][r & 3];
        if (!e_on || filter(r) >= a.F || info == 0xFFFFFFFFu) continue;
        if (THIN) {
            if ((info >> e_tap) & 1u) {
                reinterpret_cast<float *>(pout + (info >> 9))[__popc(info & ((1u << e_tap) - 1u))] = acc[0][r >> 2][r & 3];
                redo |= fabsf(acc[0][r >> 2][r & 3]) < INFINITY ? 0u : 1u << r;
            }
            continue;
        }
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        uint32_t bits = info << (32 - NT);
#pragma unroll
        for (int t = NT - 1; t >= 0; --t) {           // the four set bits of the mask, ascending
            const bool on = __builtin_uadd_overflow(bits, bits, &bits);       // (tap t's: one addition that shifts it out)
            o.w = on ? o.z : o.w; o.z = on ? o.y : o.z; o.y = on ? o.x : o.y;
            o.x = on ? acc[t][r >> 2][r & 3] : o.x;
        }
        o = make_float4(o.x * F32_UNSCALE, o.y * F32_UNSCALE, o.z * F32_UNSCALE, o.w * F32_UNSCALE);
        pout[info >> 9] = o;
        const float z = fmaf(o.x, 0.0f, fmaf(o.y, 0.0f, fmaf(o.z, 0.0f, o.w * 0.0f)));   // NaN when one of them is not finite
        redo |= z == z ? 0u : 1u << r;
    }
    // The matrix instructions multiplied the zeros around the maps and past the tile too, and 0 x Inf = NaN: these sums again,
    // over the pixels of this workgroup that exist. (Finite data pays for the check only: 8 x 32 x 32, 16 -> 16 10.3 us without, 10.5 with it;
    // 28 x 28, 128 -> 128, batch 64 78.8 and 78.7. One infinity in 1000 elements of x and of dy: that layer 3.2 ms forward, 4.9 ms here.)
    for (; redo; redo &= redo - 1u) {
        const int r = __ffs((int)redo) - 1, f = filter(r);
        const uint32_t info = kinfo[(int64_t)f * a.C + e_c], mask = info & 511u;
        constexpr int NK = THIN ? 1 : 4;          // kept taps of this lane's kernel
        int dr[NK], dc[NK];
        float sum[NK];
        uint32_t left = THIN ? 1u << e_tap : mask;
#pragma unroll
        for (int j = 0; j < NK; ++j, left &= left - 1u) {
            const int t = __ffs((int)left) - 1;
            dr[j] = t / 3 - 1;
            dc[j] = t % 3 - 1;
            sum[j] = 0.0f;
        }
        bool dead = false;                        // all NaN already
        for (int k = split; k < a.n_tiles && !dead; k += a.ksplit) {
            const int tc = k % a.tiles_c, q = k / a.tiles_c, tr = q % a.tiles_r, n = q / a.tiles_r;
            const float *dimg = dy + (int64_t)n * a.Ho * a.Wo * a.F + f, *ximg = x + (int64_t)n * a.H * a.W * a.C + e_c;
#pragma unroll 2
            for (int s = 0; s < a.TR * a.TC; ++s) {
                const int y = s / a.TC, col = s - y * a.TC, oy = tr * a.TR + y, ox = tc * a.TC + col;
                const bool on = oy < a.Ho && ox < a.Wo;
                const float d = dimg[on ? ((int64_t)oy * a.Wo + ox) * a.F : 0];
#pragma unroll
                for (int j = 0; j < NK; ++j) {
                    const int iy = oy * a.stride + dr[j], ix = ox * a.stride + dc[j];
                    const bool in = on && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
                    const float v = ximg[in ? ((int64_t)iy * a.W + ix) * a.C : 0];
                    sum[j] = in ? fmaf(d, v, sum[j]) : sum[j];
                }
            }
            dead = true;
#pragma unroll
            for (int j = 0; j < NK; ++j) dead = dead && sum[j] != sum[j];
        }
#pragma unroll
        for (int j = 0; j < NK; ++j)
            reinterpret_cast<float *>(pout + (info >> 9))[THIN ? __popc(mask & ((1u << e_tap) - 1u)) : j] = sum[j];
    }
}

pc_status pc_f32_bwd_weight(pc_ctx *ctx, const pc_conv_desc *d, const pc_packed *pk, const void *x, const void *dy, float *dw)
{
    const int64_t nslots = pk->nnzk >= 0 ? pk->nnzk : (int64_t)pk->v.F * pk->v.C;
    if (nslots == 0) return PC_OK;
    F32WgradArgs a;
    memset(&a, 0, sizeof(a));
    a.N = d->N; a.H = d->H; a.W = d->W; a.C = d->C; a.F = d->F; a.stride = d->stride;
    a.Ho = (d->H - 1) / d->stride + 1; a.Wo = (d->W - 1) / d->stride + 1;
    const bool thin = d->C <= 3;
    // The elements of x that a tile stages, and whether the staging registers hold a tile.
    auto staged_x = [&](int wc, int TR, int TC) {
        return ((TR - 1) * d->stride + 3) * (((thin ? (TC + 1) / 2 * 2 : TC) - 1) * d->stride + 3) * (thin ? 1 : 4 * wc);
    };
    auto fits = [&](int wf, int wc, int TR, int TC) {
        return TR * (thin ? (TC + 1) / 2 * 2 : TC) <= 256 * f32w_nd(wc, thin) / (8 * wf) && staged_x(wc, TR, TC) <= 256 * f32w_nx(thin);
    };
    // The tile of an arrangement of the wavefronts.
    auto tile = [&](F32WgradArgs &t, int wf, int wc, int TR, int TC) {
        const int FD = 32 * wf, CD = thin ? 4 : 16 * wc;
        t.ft = (d->F + FD - 1) / FD;
        t.ct = thin ? 1 : (d->C + CD - 1) / CD;
        t.TR = TR; t.TC = TC; t.TCe = thin ? (TC + 1) / 2 * 2 : TC;
        t.IR = (TR - 1) * d->stride + 3; t.IW = (t.TCe - 1) * d->stride + 3;
        t.nd = thin ? TR * t.TCe * (FD / 4) : 256 * f32w_nd(wc, false);     // (three parts: zeros up to the last group of 32 pixels)
        t.nx = staged_x(wc, TR, TC);
        t.tiles_r = (t.Ho + TR - 1) / TR; t.tiles_c = (t.Wo + TC - 1) / TC;
    };
    // Arrangement, pixel tile and splits by an estimate of the time (us): a start, the tiles of a workgroup (a wait, staging, matrix steps; two
    // workgroups share a CU from 256 up, two rounds from 512), the sums of wavefronts that share pixels and the pick of the kept taps, the
    // tensors' bytes, the partial planes. Fitted to 5700 timings of 160 layers (8 % rms): 3 % behind the fastest, the worst 20 % (the
    // first layer's: 10000 timings, 2.5 %; on the layers of profiles/wgrad_plan_timings_f32.csv 3.3 % and 15 %, on 12 small first layers 10 %
    // and 24 %); the widest tile that the channels fill and the pixel tile of the best throughput were 9 %
    // behind. The partial planes stay within 16 MiB. (The choice of a layer and share of kept kernels is remembered: kernel tile, pixel
    // tile, splits. Making it takes 10 to 50 us of host time.)
    int wf = 1, wc = 1, ks = 1;
    const int64_t all = (int64_t)pk->v.F * pk->v.C;
    const int share = pc_kept_share(pk);
    const int32_t key[PC_CHOICE_KEY] = {9, d->N, d->H, d->W, d->C, d->F, d->stride, share, 0, 0};
    bool known;
    int32_t *choice = pc_choice(ctx, key, &known);
    if (!known || *choice < 0) {
        const int64_t most = share ? (share * all + 31) / 32 : all;      // slots of a plane at most
        const int64_t cap = std::max((int64_t)1, ((int64_t)1 << 20) / most);
        const double kept = pc_kept_estimate(pk);
        const double moved = (thin ? 0.491e-6 : 0.466e-6) * 4.0 * ((double)a.N * a.H * a.W * a.C + (double)a.N * a.Ho * a.Wo * a.F), moved3 = moved * moved * moved;
        const double start = thin ? 6.65 : 5.0, plane0 = thin ? 2.2 : 3.5, plane = (thin ? 11.5e-6 : 14.1e-6) * kept;
        int tiles_c[65];
        for (int TC = 1; TC <= 64; ++TC) tiles_c[TC] = (a.Wo + TC - 1) / TC;
        double best = 1e30, bound = 1e30;
        *choice = -1;
        // The first walk looks at the longest tile of each number of rows and leaves a bound, which most tiles of the second exceed at once.
        for (int walk = 0; walk < 2; ++walk)
            for (int v = 0; v < 4; ++v) {
                const int vf = v & 1 ? 1 : 2, vc = v & 2 || thin ? 1 : 2, wk = 4 / (vf * vc);
                if (thin && (v & 2)) continue;
                const double end = !thin ? 0.305 : wk == 2 ? 0.39 : 1.2;
                F32WgradArgs t = a;
                tile(t, vf, vc, 1, 1);
                const int64_t T = (int64_t)t.ft * t.ct;
                int64_t splits[3];
                for (int p = 0; p < 3; ++p) splits[p] = std::min(cap, ((2 * ctx->num_cu >> p) + T - 1) / T);
                for (int TR = 1; TR <= 64 && TR <= a.Ho; ++TR) {
                    const int tiles_r = (a.Ho + TR - 1) / TR;
                    int last = 0;
                    if (walk == 0)
                        while (last < 64 && last < a.Wo && fits(vf, vc, TR, last + 1)) ++last;
                    for (int TC = walk == 0 ? std::max(1, last) : 1; TC <= 64 && TC <= a.Wo && fits(vf, vc, TR, TC); ++TC) {
                        const int TCe = thin ? (TC + 1) / 2 * 2 : TC, nd = thin ? TR * TCe * (8 * vf) : 256 * f32w_nd(vc, false);
                        const int64_t nkt = (int64_t)a.N * tiles_r * tiles_c[TC];
                        const double steps = (double)((TR * TCe / 2 + wk - 1) / wk), staged = (nd + staged_x(vc, TR, TC)) / 256.0;
                        const double lone = thin ? 0.514 + 0.0785 * steps : 1.661 + 0.106 * staged, pair = thin ? 0.618 + 0.0194 * staged + 0.117 * steps : 1.776 + 0.117 * staged;
                        // (at least one tile, and every place busy all the time, whichever the splits)
                        if (start + std::max(std::min(lone, pair), (double)nkt * (double)T / (2.0 * ctx->num_cu) * std::min(2.0 * lone, pair)) > bound) continue;
                        for (int p = 0; p < 3; ++p) {
                            const int64_t k = std::max((int64_t)1, std::min(splits[p], nkt)), G = T * k;
                            const double u = (double)((nkt + k - 1) / k);
                            const double us = start + (G <= ctx->num_cu ? u * lone + (thin ? end : 0.0) : (double)((G + 2 * ctx->num_cu - 1) / (2 * ctx->num_cu)) * (u * pair + 1.7 * end));
                            const double planes = k > 1 ? plane0 + plane * (double)k : 0.0;
                            if (std::max(us, moved) + planes > bound) continue;
                            const double c = cbrt(us * us * us + moved3) + planes;
                            if (c < bound) bound = c;
                            if (walk == 1 && c < best) {
                                best = c;
                                *choice = (vf - 1) | (vc - 1) << 1 | TR << 2 | TC << 9 | (int32_t)k << 16;
                            }
                        }
                    }
                }
            }
        if (*choice < 0) return pc_fail(ctx, PC_ERR_UNSUPPORTED, "float32 bwd_weight: no pixel tile fits");
    }
    wf = 1 + (*choice & 1); wc = 1 + (*choice >> 1 & 1); ks = *choice >> 16;
    tile(a, wf, wc, *choice >> 2 & 127, *choice >> 9 & 127);
    const int wk = 4 / (wf * wc), FD = 32 * wf, CD = thin ? 4 : 16 * wc;
    const int64_t nkt = (int64_t)a.N * a.tiles_r * a.tiles_c;
    if (nkt >= ((int64_t)1 << 31)) return pc_fail(ctx, PC_ERR_UNSUPPORTED, "float32 bwd_weight: too many pixel tiles");
    a.n_tiles = (int)nkt;
    a.mg_half = pc_udiv_magic(thin ? a.TCe / 2 : 1); a.mg_TCe = pc_udiv_magic(a.TCe); a.mg_IW = pc_udiv_magic(a.IW);
    a.pstride = nslots;
    a.ksplit = ks;
    const int64_t wgs = (int64_t)a.ft * a.ct * ks;
    a.exact = nkt * (a.tiles_c > a.tiles_r ? a.tiles_c : a.tiles_r) < ((int64_t)1 << 32) && wgs * (ks > a.ct ? ks : a.ct) < ((int64_t)1 << 32);
    a.mg_tc = pc_udiv_magic(a.tiles_c); a.mg_tr = pc_udiv_magic(a.tiles_r); a.mg_ks = pc_udiv_magic(a.ksplit); a.mg_ct = pc_udiv_magic(a.ct);
    const int planes = a.ksplit;
    void *scr = nullptr;
    if (planes > 1) {
        pc_status s = pc_scratch(ctx, sizeof(float4) * (size_t)planes * (size_t)nslots, &scr);
        if (s != PC_OK) return s;
    }
    const int PD = thin ? FD + 4 : f32w_pitch(FD), PX = thin ? 4 : f32w_pitch(CD);
    size_t lds = sizeof(float) * ((size_t)a.nd / (FD / 4) * PD + (size_t)a.IR * a.IW * PX);      // (at most 53248: the staging registers bound both)
    if (wk > 1 && lds < (size_t)(thin ? 8 : 36) * 1024) lds = (size_t)(thin ? 8 : 36) * 1024;      // in which the sums of wavefronts are added
    const dim3 grid((unsigned)(a.ft * a.ct * a.ksplit)), blk(256);
    float4 *po = planes > 1 ? (float4 *)scr : (float4 *)dw;
    const float *xp = (const float *)x, *dp = (const float *)dy;
    hipStream_t st = ctx->stream;
    const bool vec = (d->F & 3) == 0 && (d->C & 3) == 0 && (int64_t)a.H * a.W * a.C * 4 < ((int64_t)1 << 31) &&
                     (int64_t)a.Ho * a.Wo * a.F * 4 < ((int64_t)1 << 31);
    typedef void (*Kernel)(const float *, const float *, F32WgradArgs, const uint32_t *, float4 *);
    static const struct { Kernel f; int wf, wc; bool thin, vec; } kernels[] = {
#define F32W(A, B, T, V) {&pc_f32_wgrad_kernel<A, B, T, V>, A, B, T, V}
        F32W(2, 1, true, false), F32W(1, 1, true, false), F32W(2, 2, false, true), F32W(2, 2, false, false), F32W(2, 1, false, true), F32W(2, 1, false, false),
        F32W(1, 2, false, true), F32W(1, 2, false, false), F32W(1, 1, false, true), F32W(1, 1, false, false)};
#undef F32W
    int k = 0;
    while (kernels[k].wf != wf || kernels[k].wc != wc || kernels[k].thin != thin || (!thin && kernels[k].vec != vec)) ++k;
    hipLaunchKernelGGL(kernels[k].f, grid, blk, lds, st, xp, dp, a, pk->v.kinfo, po);
    pc_note_kernel(ctx, "pc_f32_wgrad_kernel<%d, %d, %s, %s>", wf, wc, thin ? "true" : "false", kernels[k].vec ? "true" : "false");
    pc_status s = pc_hip_check(ctx, hipGetLastError(), "float32 bwd_weight launch");
    if (s != PC_OK || planes == 1) return s;
    return pc_launch_wgrad_reduce(ctx, (const float *)scr, planes, nslots, nslots, pk, dw);
}
