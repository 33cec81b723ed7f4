// GEMM instances for bf16 inputs: the tiles the closed-form derivation yields
// on gfx950 (256 x 256 x 32 from LDS and registers; the CU rule's halvings
// for small problems), and the tile whose waves split K.  The last number is the
// measured time of one k position in ns, a tile per CU.
#include "gemm_ksplit_kernel.hpp"

namespace attn {

static const GemmInstance kInstances[] = {
    {ATTN_BF16, 256, 256, 32, launch_gemm<ATTN_BF16, 256, 256, 32, kGemmStages>, 24.f},
    {ATTN_BF16, 128, 256, 32, launch_gemm<ATTN_BF16, 128, 256, 32, kGemmStages>, 15.5f},
    {ATTN_BF16, 128, 128, 64, launch_gemm<ATTN_BF16, 128, 128, 64, kGemmStages>, 9.5f},
    {ATTN_BF16, 64, 128, 64, launch_gemm<ATTN_BF16, 64, 128, 64, kGemmStages>, 6.1f},
    {ATTN_BF16, 64, 64, 128, launch_gemm<ATTN_BF16, 64, 64, 128, kGemmStages>, 4.2f},
    {ATTN_BF16, 32, 64, 128, launch_gemm<ATTN_BF16, 32, 64, 128, kGemmStages>, 2.5f},
    {ATTN_BF16, kKsplitTile, kKsplitTile, kKsplitPiece, launch_gemm_ksplit<ATTN_BF16>, 1.6f},
};

const GemmInstance* gemm_instances_bf16(int* n) {
  *n = (int)(sizeof(kInstances) / sizeof(kInstances[0]));
  return kInstances;
}

}  // namespace attn
