// Count pass of the ball query (row lengths), the dispatch of the fill pass
// over dimensions, and the RDF of a stored list.
#include "pair_list.hpp"

namespace ppa {

namespace {

template <int DIM, int EXCL>
__global__ void __launch_bounds__(kBlock, 6) count_kernel(const PairIn in, const PairGeom G,
                                                       int32_t* __restrict__ counts)
{
    __shared__ float4 s_off[27];
    __shared__ StencilLds s_st[kWavesPerBlock];
    __shared__ float4 s_q[kWavesPerBlock][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uniform(threadIdx.x / kWave);
    StencilLds& S = s_st[wv];
    if (threadIdx.x < 27)
        s_off[threadIdx.x] = make_float4(G.off[threadIdx.x][0], G.off[threadIdx.x][1],
                                         G.off[threadIdx.x][2], 0.f);
    __syncthreads();
    const GeomView V = view_of(G);
    const int split = G.split > 1 ? G.split : 1;
    int t0, t1, stride;
    wave_tiles_interleaved<kWavesPerBlock>(G.ncells * split, wv, t0, t1, stride);
    for (int v = t0; v < t1; v += stride) {
        const CellPart P = cell_part(in, v, split);
        if (P.q0 == P.q1) continue;
        const int C = stencil<DIM>(in, V, P.tile, lane, S);
        count_cell<DIM, EXCL>(in, V, S, s_off, C, P.q0, P.q1, lane, s_q[wv], counts);
    }
}

__global__ void __launch_bounds__(256) hist_from_dist_kernel(const float* __restrict__ dist,
                                                             const int64_t* n_pairs,
                                                             int64_t capacity, int bins,
                                                             float r_min, float inv_dr,
                                                             unsigned long long* hist)
{
    extern __shared__ unsigned s_hist[];
    const bool lds_hist = bins <= kMaxLdsBins;
    if (lds_hist)
        for (int b = threadIdx.x; b < bins; b += blockDim.x) s_hist[b] = 0u;
    __syncthreads();
    int64_t np = *n_pairs;
    np = np < capacity ? np : capacity;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < np;
         e += (int64_t)gridDim.x * blockDim.x) {
        const float t = (dist[e] - r_min) * inv_dr;
        if (t >= 0.f && t < (float)bins) {
            const int b = min((int)t, bins - 1);
            if (lds_hist)
                atomicAdd(&s_hist[b], 1u);
            else
                atomicAdd(&hist[b], 1ull);
        }
    }
    __syncthreads();
    if (lds_hist)
        for (int b = threadIdx.x; b < bins; b += blockDim.x) {
            const unsigned v = s_hist[b];
            if (v) atomicAdd(&hist[b], (unsigned long long)v);
        }
}

template <int DIM, int EXCL>
void launch_count_t(const PairIn& in, const PairGeom& g, int32_t* counts, hipStream_t s)
{
    auto k = count_kernel<DIM, EXCL>;
    const int blocks = resident_blocks(k, 0, (long long)g.ncells * (g.split > 1 ? g.split : 1));
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), 0, s, in, g, counts);
}

}  // namespace

void launch_count(const PairArgs& a, int dim, int excl, hipStream_t s)
{
    const PairIn in = make_in(a);
#define PPA_COUNT(D, E) launch_count_t<D, E>(in, a.geom, a.counts, s)
    if (dim == 3) {
        if (excl == 1) PPA_COUNT(3, 1); else if (excl == 2) PPA_COUNT(3, 2); else PPA_COUNT(3, 0);
    } else {
        if (excl == 1) PPA_COUNT(2, 1); else if (excl == 2) PPA_COUNT(2, 2); else PPA_COUNT(2, 0);
    }
#undef PPA_COUNT
}

void launch_fill(const PairArgs& a, int dim, int excl, bool nl, bool hist, hipStream_t s)
{
    if (dim == 3)
        launch_fill_3d(a, excl, nl, hist, s);
    else
        launch_fill_2d(a, excl, nl, hist, s);
}

void launch_hist_from_dist(const float* dist, const int64_t* n_pairs, int64_t capacity, int bins,
                           float r_min, float inv_dr, unsigned long long* hist, hipStream_t s)
{
    const size_t lds = bins <= kMaxLdsBins ? sizeof(unsigned) * (size_t)bins : 0;
    hipLaunchKernelGGL(hist_from_dist_kernel, dim3(1024), dim3(256), lds, s, dist, n_pairs,
                       capacity, bins, r_min, inv_dr, hist);
}

}  // namespace ppa
