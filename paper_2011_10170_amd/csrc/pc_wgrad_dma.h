// Backward-weight with operands straight from NHWC rows in LDS: launch description (pc_wgrad_dma.hip).
#ifndef PC_WGRAD_DMA_H
#define PC_WGRAD_DMA_H
#include "pc_mfma.h"

#define WD_LDS_MAX (80 * 1024)       // two workgroups per CU
#define WD_GROUP_MAX 20

struct WgradDmaArgs {
    int32_t N, H, W, C, F, Ho, Wo, stride;
    int32_t rows;                    // N * Ho
    int32_t TR, TC, IW, nrow;        // rows (a multiple of 16) and columns of a pixel tile, staged x columns and rows
    int32_t RPx, RPd, dy_off;        // bytes per staged row of x and dy, LDS offset of dy
    int32_t tiles_c, n_ktiles, ksplit, pstride;
    uint32_t x_bytes, dy_bytes;
    uint32_t mg_tc, mg_Ho, mg_H1;
};

struct WgradDmaLayer {
    WgradDmaArgs a;
    const uint16_t *x, *dy;
    const uint32_t *kinfo;
    float *partial, *dw;
    int32_t gx, gy;
};

struct WgradDmaGroup {
    int32_t n;
    int32_t blk0[WD_GROUP_MAX + 1];
    WgradDmaLayer layer[WD_GROUP_MAX];
};

// Plan of one layer (ksplit left to the caller); false when the layer is outside what the kernel takes. *tile_us: estimated time of a
// pixel tile (us) while two workgroups share a CU.
bool pc_wgrad_dma_plan(const pc_conv_desc *d, int64_t nslots, WgradDmaArgs *out, int *ct, int *ft, size_t *lds, double *tile_us);
pc_status pc_wgrad_dma_launch(pc_ctx *ctx, const WgradDmaGroup &g, size_t lds);
#endif
