// Fill pass of the ball query, 2D.
#include "fill_kernel.hpp"

namespace ppa {

void launch_fill_2d(const PairArgs& a, int excl, bool nl, bool hist, hipStream_t s)
{
    launch_fill_dim<2>(a, excl, nl, hist, s);
}

}  // namespace ppa
