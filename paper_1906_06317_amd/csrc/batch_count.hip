// Count pass of a batch (row lengths of every frame).
#include "batch_queue.hpp"

namespace ppa {

namespace {

// Row lengths of a batch; WPB wavefronts per workgroup.
template <int DIM, int EXCL, int WPB>
__global__ void __launch_bounds__(WPB * kWave, 5) count_batch_kernel(
    const PairIn in, const BatchGeom B, int32_t* __restrict__ counts)
{
    __shared__ float4 s_off[WPB][27];
    __shared__ StencilLds s_st[WPB];
    __shared__ float4 s_q[WPB][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uniform(threadIdx.x / kWave);
    StencilLds& S = s_st[wv];
    float4* off = s_off[wv];
    RunQueue<8> R;
    R.start(B, WPB, wv);
    const FrameSearch frames(B, lane);
    int f = -1, cur = 0, next = -1;
    GeomView V;
    int t, te;
    while (R.next(B, B.queue, lane, t, te)) {
        for (int v = t; v < te; ++v) {
            const CellPart P = cell_part(in, v, B.split);
            if (P.q0 == P.q1) continue;
            if (P.tile < cur || P.tile >= next) {
                f = frames.find(B, P.tile, lane);
                cur = B.cell_base[f];
                next = B.cell_base[f + 1];
                V = load_frame(B, f, off, lane);
            }
            const int C = stencil<DIM>(in, V, P.tile, lane, S);
            count_cell<DIM, EXCL>(in, V, S, off, C, P.q0, P.q1, lane, s_q[wv], counts);
        }
    }
}

template <int DIM, int EXCL, int WPB>
void count_batch_t(const PairIn& in, const BatchGeom& b, int32_t* counts, int blocks_cap,
                          hipStream_t s)
{
    auto k = count_batch_kernel<DIM, EXCL, WPB>;
    const int blocks = batch_blocks(k, WPB * kWave, 0, blocks_cap);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(WPB * kWave), 0, s, in, b, counts);
}

}  // namespace

void launch_count_batch(const PairArgs& a, const BatchGeom& b, int dim, int excl, int blocks_cap,
                        int waves, hipStream_t s)
{
    const PairIn in = make_in(a);
#define PPA_CB(D, E)                                                         \
    do {                                                                     \
        if (waves == 2) count_batch_t<D, E, 2>(in, b, a.counts, blocks_cap, s); \
        else count_batch_t<D, E, 4>(in, b, a.counts, blocks_cap, s);        \
    } while (0)
    if (dim == 3) {
        if (excl) PPA_CB(3, 1); else PPA_CB(3, 0);
    } else {
        if (excl) PPA_CB(2, 1); else PPA_CB(2, 0);
    }
#undef PPA_CB
}

void launch_fill_batch(const PairArgs& a, const BatchGeom& b, int dim, int excl, int blocks_cap,
                       int waves, hipStream_t s)
{
    if (dim == 3)
        launch_fill_batch_3d(a, b, excl, blocks_cap, waves, s);
    else
        launch_fill_batch_2d(a, b, excl, blocks_cap, waves, s);
}

}  // namespace ppa
