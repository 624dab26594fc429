// fp32-storage instantiations of the forward kernel for many maps, eight channels per workgroup (scan2d_fwd_quads.hpp).
#include "scan2d_variants.hpp"
#include "scan2d_fwd_quads.hpp"
namespace scan2d {
FwdKernel fwd_quads_kernel_f32(int K, bool sp, bool gate) { return lookup_fwd_quads_kernel<float>(K, sp, gate); }
}
