// bf16-storage instantiations of the forward kernel for many maps, eight channels per workgroup (scan2d_fwd_quads.hpp).
#include "scan2d_variants.hpp"
#include "scan2d_fwd_quads.hpp"
namespace scan2d {
FwdKernel fwd_quads_kernel_bf16(int K, bool sp, bool gate) { return lookup_fwd_quads_kernel<bf16_t>(K, sp, gate); }
size_t fwd_quads_lds(int K, int cols) {
#define SCAN2D_X(k) if (K == k) return quad_lds_bytes<k>(cols);
    SCAN2D_FWD_QUADS_COLUMNS(SCAN2D_X)
#undef SCAN2D_X
    return 0;
}
}
