// Fill pass of a batch (NeighborList and per-frame RDF); included once per
// dimension.
#pragma once

#include "batch_queue.hpp"

namespace ppa {

namespace {

// Adds this wavefront's LDS histogram into the global one and clears it.
__device__ __forceinline__ void merge_wave_hist(unsigned* h, unsigned long long* g, int bins,
                                                int lane)
{
    wave_sync();
    for (int b = lane; b < bins; b += kWave) {
        const unsigned v = h[b];
        if (v) {
            atomicAdd(&g[b], (unsigned long long)v);
            h[b] = 0u;
        }
    }
    wave_sync();
}

// Rows buffered per wavefront in a batch.  The workgroup's LDS (with a
// histogram per wavefront) decides how many share a CU: it is handed out in
// units of 1280 bytes, so five fit up to 32,000.  At 64 rows and 128 bins
// it was 128 bytes over, a fifth of the persistent workgroups began only when
// others had ended; 40 rows (which bind only below eight hits a row) fit up to
// 256 bins: 556 -> 536 us for 96 frames, 62 M pairs.
constexpr int kBatchRows = 40;

// NeighborList and per-frame RDF (histograms [nframes][bins]) of a batch;
// WPB wavefronts per workgroup.
template <int DIM, int EXCL, int WPB>
__global__ void __launch_bounds__(WPB * kWave, 5) fill_batch_kernel(
    const PairIn in, const BatchGeom B, const FillOut O)
{
    extern __shared__ unsigned s_dyn[];  // one histogram per wavefront when bins are few
    __shared__ float4 s_off[WPB][27];
    __shared__ FillLds<true, kBatchRows> s_w[WPB];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uniform(threadIdx.x / kWave);
    StencilLds& S = s_w[wv].st;
    float4* off = s_off[wv];
    const bool lds_hist = O.bins <= kMaxBatchLdsBins;
    unsigned* h = lds_hist ? s_dyn + (size_t)wv * O.bins : nullptr;
    if (lds_hist)
        for (int b = lane; b < O.bins; b += kWave) h[b] = 0u;
    if (lane < kHitCap / 64) s_w[wv].starts[lane] = 0ull;
    wave_sync();
    Filler<DIM, EXCL, true, true, kBatchRows> F(s_w[wv], O, h, lane);
    RunQueue<32> R;
    unsigned long long* queue = B.queue + 8 * kQueueStride;
    R.start(B, WPB, wv);
    const FrameSearch frames(B, lane);
    int f = -1, cur = 0, next = -1;
    GeomView V;
    int t, te;
    while (R.next(B, queue, lane, t, te)) {
        for (int v = t; v < te; ++v) {
            const CellPart P = cell_part(in, v, B.split);
            if (P.q0 == P.q1) continue;
            if (P.tile < cur || P.tile >= next) {
                // buffered hits belong to the old frame: write them and its bins first
                if (F.nh > 0) F.flush();
                if (lds_hist && f >= 0) merge_wave_hist(h, F.ghist, O.bins, lane);
                f = frames.find(B, P.tile, lane);
                cur = B.cell_base[f];
                next = B.cell_base[f + 1];
                V = load_frame(B, f, off, lane);
                F.ghist = O.hist + (size_t)f * O.bins;
                F.id_base = uniform(B.frames[f].point_base);
            }
            const int C = stencil<DIM>(in, V, P.tile, lane, S);
            const int ns = (C + kWave - 1) / kWave;
            switch (ns) {
#define PPA_CASE(N)                                                                         \
    case N: fill_tile<DIM, EXCL, true, true, N>(in, V, S, off, C, P.qc, P.q0, P.q1, F); \
        break;
                PPA_CASE(0) PPA_CASE(1) PPA_CASE(2) PPA_CASE(3) PPA_CASE(4) PPA_CASE(5)
                PPA_CASE(6) PPA_CASE(7) PPA_CASE(8) PPA_CASE(9) PPA_CASE(10)
#undef PPA_CASE
            default: fill_chunked<DIM, EXCL, true, true>(in, V, S, off, C, P.q0, P.q1, F);
            }
        }
    }
    if (F.nh > 0) F.flush();
    if (lds_hist && f >= 0) merge_wave_hist(h, F.ghist, O.bins, lane);
    if (__ballot(F.over) && lane == 0) atomicOr(O.status, kStatusCapacity);
}

template <int DIM, int EXCL, int WPB>
void fill_batch_t(const PairIn& in, const BatchGeom& b, const FillOut& o, int blocks_cap,
                         hipStream_t s)
{
    const size_t lds =
        o.bins <= kMaxBatchLdsBins ? sizeof(unsigned) * (size_t)o.bins * WPB : 0;
    auto k = fill_batch_kernel<DIM, EXCL, WPB>;
    const int blocks = batch_blocks(k, WPB * kWave, lds, blocks_cap);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(WPB * kWave), lds, s, in, b, o);
}

template <int DIM>
void launch_fill_batch_dim(const PairArgs& a, const BatchGeom& b, int excl, int blocks_cap,
                           int waves, hipStream_t s)
{
    const PairIn in = make_in(a);
    const FillOut o = make_out(a, true);
    if (waves == 2) {
        if (excl)
            fill_batch_t<DIM, 1, 2>(in, b, o, blocks_cap, s);
        else
            fill_batch_t<DIM, 0, 2>(in, b, o, blocks_cap, s);
    } else {
        if (excl)
            fill_batch_t<DIM, 1, 4>(in, b, o, blocks_cap, s);
        else
            fill_batch_t<DIM, 0, 4>(in, b, o, blocks_cap, s);
    }
}

}  // namespace

}  // namespace ppa
