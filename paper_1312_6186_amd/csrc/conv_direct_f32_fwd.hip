// conv_direct_kernel for f32, bias + ReLU epilogue.
#include "conv_direct.h"

namespace asgd {

int launch_direct_f32_fwd(int tile, int ks, const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s)
{
    return launch_direct_t<float, false>(tile, ks, p, ep, grid, lds, s);
}

}  // namespace asgd
