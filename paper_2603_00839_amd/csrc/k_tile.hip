// Tile kernel (the stage itself is tile_task in tile_body.h).
#include "tile_body.h"

namespace rtg {

// Four float32 sketch tiles per wave take 296 registers with blocks of 256 rows:
// one workgroup per compute unit.  Where three are enough (sketches of 65 to 96
// rows) they are bounded to the registers of two: 12 problems of 712x500x3 with
// 89 sketch rows (576 column tiles, m = 12) 2.96 -> 2.62 ms.  Four bounded to
// the same spill a little, which costs 1 % where many terms are read (64 uneven
// images, m = 40: 16.7 ms in this kernel, 16.9 bounded); the forms with two fit
// by themselves, and the bound cost Golub-Kahan's 64-row blocks 1 %.  The
// two-plane form's 64-row blocks fit three workgroups only when bounded to them.
template <bool BB, bool MB, bool SPLIT, int RPW, int SBR>
__global__ void __launch_bounds__(256, RPW == 3 ? 2 : (SPLIT && RPW == 2 && SBR == 64 ? 3 : 1)) k_tile(const Desc* __restrict__ descs,
                                              const int* __restrict__ starts, int count,
                                              int mode, int nterms_arg, int dst_index, int t0) {
    __shared__ TileShared<MB, SPLIT, RPW, SBR> sh;
    tile_task<BB, MB, SPLIT, RPW, SBR>(descs, starts, count, mode, nterms_arg, dst_index, t0, blockIdx.x, sh);
}

hipError_t launch_tile(const Desc* d, const int* starts, int count, int total_tiles, int mode,
                       int nterms, int dst_index, int basis_bf16, int src_bf16, int l1max, hipStream_t s,
                       int first_term, int rows, int sketch_bf16, int block_rows, int composed) {
#define RTG_TILE_B(BBV, MBV, SPV, RPV, SBV)                                                       \
    hipLaunchKernelGGL((k_tile<BBV, MBV, SPV, RPV, SBV>), dim3(total_tiles), dim3(256), 0, s, d, starts, count, \
                       mode, nterms, dst_index, first_term)
#define RTG_TILE(BBV, MBV, SPV, RPV)                                         \
    do {                                                                     \
        if (block_rows <= 64) RTG_TILE_B(BBV, MBV, SPV, RPV, 64);            \
        else if (block_rows <= 128) RTG_TILE_B(BBV, MBV, SPV, RPV, 128);     \
        else RTG_TILE_B(BBV, MBV, SPV, RPV, 256);                            \
    } while (0)
    const bool newv = mode == TM_NEWV || mode == TM_GKNEW || mode == TM_NEWV1;
    const int rtiles = ((l1max + 15) / 16) * (newv && composed ? 2 : 1);
    const bool small = rtiles <= 8 && rows != 4;
    const bool split = (mode == TM_SKETCH_SRC || mode == TM_SKETCH_W) && !src_bf16;
    if (basis_bf16) {
        if (split) { if (small) RTG_TILE(true, true, true, 2); else RTG_TILE(true, true, true, 4); }
        else { if (small) RTG_TILE(true, true, false, 2); else RTG_TILE(true, true, false, 4); }
    } else if (sketch_bf16) {
        // float32 basis with bfloat16 products: sources that are not a basis
        // tensor (R0, W) keep the two-plane split, new basis tensors one plane
        if (split) { if (small) RTG_TILE(false, true, true, 2); else RTG_TILE(false, true, true, 4); }
        else { if (small) RTG_TILE(false, true, false, 2); else RTG_TILE(false, true, false, 4); }
    } else {
        if (small) RTG_TILE(false, false, false, 2);
        else if (rtiles <= 12 && rows != 4) RTG_TILE(false, false, false, 3);
        else RTG_TILE(false, false, false, 4);
    }
#undef RTG_TILE
#undef RTG_TILE_B
    return hipGetLastError();
}

}  // namespace rtg
