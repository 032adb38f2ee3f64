// Fill pass of the ball query for one frame (list, list with RDF, or RDF
// alone); included once per dimension.
#pragma once

#include "pair_list.hpp"

namespace ppa {

namespace {

// The queries of one work item: the slot count picks the unrolled code.
template <int DIM, int EXCL, bool NL, bool HIST>
__device__ __forceinline__ void fill_cell(const PairIn& in, const GeomView& V, StencilLds& S,
                                          const float4* s_off, const CellPart P,
                                          Filler<DIM, EXCL, NL, HIST>& F)
{
    if (P.q0 == P.q1) return;
    const int C = stencil<DIM>(in, V, P.tile, F.lane, S);
    const int ns = (C + kWave - 1) / kWave;
    switch (ns) {
#define PPA_CASE(N)                                                                    \
    case N: fill_tile<DIM, EXCL, NL, HIST, N>(in, V, S, s_off, C, P.qc, P.q0, P.q1, F); \
        break;
        PPA_CASE(0) PPA_CASE(1) PPA_CASE(2) PPA_CASE(3) PPA_CASE(4) PPA_CASE(5) PPA_CASE(6)
        PPA_CASE(7) PPA_CASE(8) PPA_CASE(9) PPA_CASE(10)
#undef PPA_CASE
        static_assert(kFillSlots == 10, "the cases above cover 0..kFillSlots");
    default: fill_chunked<DIM, EXCL, NL, HIST>(in, V, S, s_off, C, P.q0, P.q1, F);
    }
}

template <int DIM, int EXCL, bool NL, bool HIST>
__global__ void __launch_bounds__(kBlock, 5) fill_kernel(const PairIn in, const PairGeom G,
                                                      const FillOut O)
{
    extern __shared__ unsigned s_hist[];
    __shared__ float4 s_off[27];
    __shared__ FillLds<NL> s_w[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uniform(threadIdx.x / kWave);
    StencilLds& S = s_w[wv].st;
    const bool lds_hist = HIST && O.bins <= kMaxLdsBins;
    if (threadIdx.x < 27)
        s_off[threadIdx.x] = make_float4(G.off[threadIdx.x][0], G.off[threadIdx.x][1],
                                         G.off[threadIdx.x][2], 0.f);
    if (lds_hist)
        for (int b = threadIdx.x; b < O.bins; b += kBlock) s_hist[b] = 0u;
    __syncthreads();

    if constexpr (NL) {
        if (lane < kHitCap / 64) s_w[wv].starts[lane] = 0ull;
        wave_sync();
    }
    Filler<DIM, EXCL, NL, HIST> F(s_w[wv], O, lds_hist ? s_hist : nullptr, lane);
    const GeomView V = view_of(G);
    const int split = G.split > 1 ? G.split : 1;
    const int items = G.ncells * split;
    if constexpr (NL || DIM == 2) {
        CellWalk<kWavesPerBlock> walk(items, wv, lane, G.dealt, G.queue);
        for (int v; walk.next(v);)
            fill_cell<DIM, EXCL, NL, HIST>(in, V, S, s_off, cell_part(in, uniform(v), split), F);
    } else {
        // every cell dealt, as the walk would (2^20 points, 7 neighbours, whole call: 218 us in 3D,
        // 225 by the walk; in 2D the walk is the faster one, 179 us and 190)
        int t0, t1, stride;
        wave_tiles_interleaved<kWavesPerBlock>(items, wv, t0, t1, stride);
        for (int v = t0; v < t1; v += stride)
            fill_cell<DIM, EXCL, NL, HIST>(in, V, S, s_off, cell_part(in, v, split), F);
    }
    if (F.nh > 0) F.flush();
    if (NL && __ballot(F.over) && lane == 0) atomicOr(O.status, kStatusCapacity);
    if (!NL && EXCL == 1 && F.selfs > 0 && O.r_min <= 0.f && lane == 0) {
        if (lds_hist)
            atomicSub(&s_hist[0], (unsigned)F.selfs);
        else
            atomicAdd(&O.hist[0], (unsigned long long)(-(long long)F.selfs));
    }

    __syncthreads();
    if (lds_hist)
        for (int b = threadIdx.x; b < O.bins; b += kBlock) {
            const unsigned v = s_hist[b];
            if (v) atomicAdd(&O.hist[b], (unsigned long long)v);
        }
}

template <int DIM, int EXCL>
void launch_fill_t(const PairIn& in, const PairGeom& g, const FillOut& o, bool nl, bool hist,
                   hipStream_t s)
{
    const size_t lds = (hist && o.bins <= kMaxLdsBins) ? sizeof(unsigned) * (size_t)o.bins : 0;
    auto k = nl ? (hist ? fill_kernel<DIM, EXCL, true, true> : fill_kernel<DIM, EXCL, true, false>)
                : fill_kernel<DIM, EXCL, false, true>;
    const long long items = (long long)g.ncells * (g.split > 1 ? g.split : 1);
    const int blocks = resident_blocks(k, lds, items);
    PairGeom geom = g;
    geom.dealt = g.draw ? dealt_rounds(items, blocks, kWavesPerBlock) : -1;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), lds, s, in, geom, o);
}

template <int DIM>
void launch_fill_dim(const PairArgs& a, int excl, bool nl, bool hist, hipStream_t s)
{
    const PairIn in = make_in(a);
    const FillOut o = make_out(a, hist);
    if (excl == 1)
        launch_fill_t<DIM, 1>(in, a.geom, o, nl, hist, s);
    else if (excl == 2)
        launch_fill_t<DIM, 2>(in, a.geom, o, nl, hist, s);
    else
        launch_fill_t<DIM, 0>(in, a.geom, o, nl, hist, s);
}

}  // namespace

}  // namespace ppa
