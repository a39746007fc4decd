// conv_direct_kernel for bf16, bias + ReLU epilogue.
#include "conv_direct.h"

namespace asgd {

int launch_direct_bf16_fwd(int tile, int ks, const DirectConv &p, const Epilogue &ep, unsigned grid, unsigned lds, hipStream_t s)
{
    return launch_direct_t<bf16_t, false>(tile, ks, p, ep, grid, lds, s);
}

}  // namespace asgd
