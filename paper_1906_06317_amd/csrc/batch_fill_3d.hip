// Fill pass of a batch, 3D.
#include "batch_fill_kernel.hpp"

namespace ppa {

void launch_fill_batch_3d(const PairArgs& a, const BatchGeom& b, int excl, int blocks_cap,
                           int waves, hipStream_t s)
{
    launch_fill_batch_dim<3>(a, b, excl, blocks_cap, waves, s);
}

}  // namespace ppa
