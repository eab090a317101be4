// Backward-weight with operands straight from NHWC rows in LDS: launch description (pc_wgrad_dma.hip).
#ifndef PC_WGRAD_DMA_H
#define PC_WGRAD_DMA_H
#include "pc_mfma.h"

#define WD_LDS_MAX (80 * 1024)       // two workgroups per CU
#define WD_LDS_SUMS (4 * 18 * 1024)  // in which wavefronts that share pixels add their sums
#define WD_GROUP_MAX 20
#define WD_WAVES 4                   // arrangements of a workgroup's wavefronts

struct WgradDmaArgs {
    int32_t N, H, W, C, F, Ho, Wo, stride;
    int32_t rows;                    // N * Ho
    int32_t TR, TC, IW, nrow;        // rows (a multiple of 16) and columns of a pixel tile, staged x columns and rows
    int32_t RPx, RPd, dy_off;        // bytes per staged row of x and dy, LDS offset of dy
    int32_t tiles_c, n_ktiles, ksplit, pstride;
    uint32_t x_bytes, dy_bytes;
    uint32_t mg_tc, mg_Ho, mg_H1;
    int32_t waves, lgPC, NC;         // arrangement of the wavefronts; of those that share pixels side by side (log2), each with NC columns
    // set at the launch: tiles of the layer, and how a workgroup's index is read, so that those of an XCD share as few pixel splits as possible
    int32_t T, place, lgks;
    uint32_t mg_T, mg_gx;
};
enum { WD_PLACE_PLAIN, WD_PLACE_MANY, WD_PLACE_FEW };

struct WgradDmaLayer {
    WgradDmaArgs a;
    const uint16_t *x, *dy;
    const uint32_t *kinfo;
    float *partial, *dw;
    int32_t gx, gy;
};

// A layer with at most 4 input channels.
struct ThinWgradArgs {
    int32_t N, H, W, C, F, Ho, Wo, stride;
    int32_t rows, TC, IW, nx;        // N * Ho; columns of a tile, staged x columns and pixels
    int32_t RPx, RPd, x_off, buf_bytes;
    int32_t tiles_c, n_tiles, pstride;
    uint32_t x_bytes, dy_bytes;
    uint32_t mg_tc, mg_Ho, mg_H1, mg_IW;
};
struct ThinWgradLayer {
    ThinWgradArgs a;
    const uint16_t *x, *dy;
    const uint32_t *kinfo;
    float *out;
    int32_t ksplit, blocks_f;             // ksplit = 0: none
};

template <int LAYERS> struct WgradDmaLayers {
    int32_t n;
    int32_t blk0[WD_GROUP_MAX + 1];
    WgradDmaLayer layer[LAYERS];
};
typedef WgradDmaLayers<1> WgradDmaOne;
struct WgradDmaGroup : WgradDmaLayers<WD_GROUP_MAX> { ThinWgradLayer thin; };
static_assert(sizeof(WgradDmaOne) == 272 && sizeof(WgradDmaGroup) <= 4096, "kernel arguments");

struct WgradDmaPlan {
    WgradDmaArgs a;
    int ct, ft;                      // tiles of channels and of filters
    int steps, loads;                // of a pixel tile: steps of 36 matrix instructions and direct loads per wavefront
    size_t lds;
    double tile_us, end_us;          // estimated time of a pixel tile (us) while two workgroups share a CU, and of a workgroup's end
    double us;                       // plan_one, not of a remembered choice: of the layer
};

// Plan of one layer of a grouped call (ksplit left to the caller), and of a layer's own call; false when the layer is outside what the kernel
// takes. kept: kernels whose partial sums are written and read; waves: the arrangement to take, -1 = any; *choice: the plan made before
// for this layer, or -1 and the plan's code on return (plan_one: may be null).
bool pc_wgrad_dma_plan(const pc_conv_desc *d, int64_t nslots, int32_t *choice, WgradDmaPlan *out);
bool pc_wgrad_dma_plan_one(const pc_conv_desc *d, int64_t nslots, double kept, int num_cu, int waves, int32_t *choice, WgradDmaPlan *out);
pc_status pc_wgrad_dma_launch(pc_ctx *ctx, WgradDmaOne &g, size_t lds);
pc_status pc_wgrad_dma_launch(pc_ctx *ctx, WgradDmaGroup &g, size_t lds);

// A layer of few pixels in one launch, without scratch: the tile (16 x 16, 16 x 32, 32 x 16, 32 x 32 filters x channels) of the least estimated
// time below limit (us) or -1, and its launch.
int pc_wgrad_few_tile(const pc_conv_desc *d, int num_cu, double limit);
pc_status pc_mfma_bwd_weight_few(pc_ctx *ctx, const pc_conv_desc *d, const pc_packed *pk, const void *x, const void *dy, float *dw, int tile, bool *launched);

struct ThinWgradPlan {
    ThinWgradArgs a;
    int nf, xp, blocks_f, ksplit;    // blocks of 16 filters per workgroup, pixels of x per thread, blocks of 64 filters, workgroups that share the tiles
    size_t lds;
};
bool pc_thin_wgrad_plan(const pc_conv_desc *d, int64_t nslots, int num_cu, ThinWgradPlan *out);
pc_status pc_thin_wgrad_launch(pc_ctx *ctx, const ThinWgradPlan &p, const uint16_t *x, const uint16_t *dy, const uint32_t *kinfo, float *out);
#endif
