// Gaussian-smoothed RDF and its adjoint (an extension beyond the paper: a
// differentiable form of the density module's RDF).
//
//   phi(u) = exp(-u^2 / (2 s^2)) / (s sqrt(2 pi)),   c_b = (b + 1/2) dr,
//   h_b    = dr * sum over ordered pairs (i, j), i != j, r_ij < r_max + 8 s,
//            of phi(c_b - r_ij) for the bins with |c_b - r_ij| <= 8 s;
//   given G_b = dL/dh_b:
//   dL/dp_k = sum over j != k of 2 A(r_kj) (p_k - p_j) / r_kj,
//   A(r)    = sum_b G_b dr (c_b - r) / s^2 phi(c_b - r)   (same window),
// the factor 2 collecting the pairs (k, j) and (j, k); a pair at r = 0
// contributes nothing to the gradient.
//
// Both passes find their pairs over the cell list (cells of width >= r_max
// + 8 s, one wavefront per home cell, candidates in register slots tested
// in float32) and compact the hits into a per-wavefront LDS buffer as
// (candidate position in the sorted array, stencil slot, query lane).  At
// the flush every lane takes one hit and recomputes its pair vector in
// float64 from the stored cell-local coordinates and a float64 stencil
// offset, so the distance entering the Gaussian is exact to the rounding of
// the stored coordinates; the window terms are then evaluated in float32
// with the hardware exp2.  The forward adds each term into a float64 LDS
// histogram per workgroup (partials summed by a second kernel); the adjoint
// gathers each query's row in float64, so every particle's gradient is
// written once, by the wavefront that owns it, with no atomics.  For given
// G, A(r) is one smooth function of r for every pair: a small kernel tabulates
// it with three derivatives at nodes sigma / 64 apart (Hermite functions of
// the window terms, summed in float64), and a pair takes one 16-byte read and
// a cubic instead of its window's terms.  The adjoint recomputes the pairs
// instead of reading anything stored by the forward.
#include "pair_common.hpp"

namespace ppa {

namespace {

using namespace pair;

constexpr int kSmSlots = 8;   // candidate slots per chunk
constexpr int kSmBuf = 768;   // hits buffered per wavefront
constexpr int kSmFlushAt = kSmBuf - kSmSlots * kWave;

template <int BUF>
struct SmoothLds {
    int2 hit[BUF];  // (sorted candidate index, stencil slot | query lane << 5)
    float4 q[kWave];   // the query chunk: cell-local xyz, index bits
    StencilLds st;
};

// The forward is bound by its float64 LDS atomics (about 1.4 lanes a clock per CU
// whatever the addresses) and by vector issue: 131,072 points, 21 bins a
// window, 374 us.  Two 20-bit limbs of a fixed-point sum by 32-bit atomics took 340 us,
// but keep a term's 24 bits only down to 2^-17 of the largest one: 5.6e-5 off at
// 5 sigma and nothing left past 7.4.  With float64 sums for the smaller terms, or with
// three pairs of limbs 17 bits apart, both exact, the whole call took 440 us instead of 415.
template <int BUF>
struct SmoothShared {
    float4 off[27];
    double offd[27][3];
    SmoothLds<BUF> w[kWavesPerBlock];
};

// Candidates [k0, k0 + 64 NS) of a stencil: coordinates relative to the
// home cell's centre in float32 (for the cut), sorted index and slot.
template <int DIM, int NS>
struct SmSlots {
    float x[NS], y[NS], z[NS];
    int idx[NS];  // sorted position; -1 past the end
    int j[NS];    // stencil slot

    __device__ __forceinline__ void load(const PairIn& in, const PairGeom& G, const StencilLds& S,
                                         const float4* off, int k0, int C, int lane)
    {
        int before = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            x[s] = y[s] = z[s] = kFar;
            idx[s] = -1;
            j[s] = 0;
            const int k = k0 + s * kWave + lane;
            const int jj = cell_of(S, G.nsten, k0, s, k, C, before);
            if (k < C) {
                const int p = S.base[jj] + k;
                const float4 v = in.cand[p];
                const float4 o = off[jj];
                x[s] = v.x + o.x;
                y[s] = v.y + o.y;
                z[s] = DIM == 3 ? v.z + o.z : 0.f;
                idx[s] = p;
                j[s] = jj;
            }
        }
    }
};

// Pair vector of a buffered hit in float64, candidate minus query.
template <int DIM, int BUF>
__device__ __forceinline__ void hit_vector(const SmoothArgs& a, const SmoothShared<BUF>& L,
                                           const SmoothLds<BUF>& W, int2 h, double& dx, double& dy,
                                           double& dz)
{
    const int j = h.y & 31;
    const float4 v = a.cand[h.x];
    const float4 q = W.q[h.y >> 5];
    dx = ((double)v.x - (double)q.x) + L.offd[j][0];
    dy = ((double)v.y - (double)q.y) + L.offd[j][1];
    dz = DIM == 3 ? ((double)v.z - (double)q.z) + L.offd[j][2] : 0.0;
}

// Bins of the window around r: |c_b - r| <= 8 s, inside [0, bins).  The
// bounds are found in float32 (a bin at the edge carries weight e^-32, so
// where rounding puts the edge does not matter); the offset of the first
// bin centre from r is exact to float64 before rounding.
__device__ __forceinline__ void window(const SmoothArgs& a, double r, int& b0, int& b1, float& u0)
{
    const float rf = (float)r, w8 = (float)a.w8;
    b0 = max(0, (int)ceilf(fmaf(rf - w8, a.inv_dr, -0.5f)));
    b1 = min(a.bins - 1, (int)floorf(fmaf(rf + w8, a.inv_dr, -0.5f)));
    u0 = (float)fma((double)b0 + 0.5, a.dr, -r);
}

// Hits of query t (scalar) against NS slots, appended to the buffer.
template <int DIM, int NS, int BUF>
__device__ __forceinline__ int buffer_query(const SmSlots<DIM, NS>& c, SmoothLds<BUF>& W, int nh,
                                            float qx, float qy, float qz, int qpos, int t,
                                            float r2s, int left)
{
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s * kWave >= left) break;  // the last chunk may leave slots empty
        const bool h = dist2<DIM>(c.x[s] - qx, c.y[s] - qy, c.z[s] - qz) < r2s && c.idx[s] != qpos;
        const unsigned long long m = __ballot(h);
        if (h) W.hit[nh + (int)lane_prefix(m)] = make_int2(c.idx[s], c.j[s] | (t << 5));
        nh += __popcll(m);
    }
    return nh;
}

// Forward flush: every buffered pair's window terms into the LDS histogram.
template <int DIM, int BUF>
__device__ __forceinline__ void flush_fwd(const SmoothArgs& a, const SmoothShared<BUF>& L,
                                          SmoothLds<BUF>& W, double* hist, int nh, int lane)
{
    wave_sync();
    const float drf = (float)a.dr;
    for (int e = lane; e < nh; e += kWave) {
        double dx, dy, dz;
        hit_vector<DIM, BUF>(a, L, W, W.hit[e], dx, dy, dz);
        const double r = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
        int b0, b1;
        float u0;
        window(a, r, b0, b1, u0);
        // each lane starts its walk at a different bin of its window, so the
        // lanes of one instruction rarely add to the same bin
        const int nb = b1 - b0 + 1;
        int m = nb > 0 ? lane % nb : 0;
#pragma unroll 4
        for (int j = 0; j < nb; ++j) {
            const float u = fmaf((float)m, drf, u0);
            const float v = a.hscale * __builtin_amdgcn_exp2f(-(u * u) * a.k2);
            atomicAdd(&hist[b0 + m], (double)v);
            m = m + 1 == nb ? 0 : m + 1;
        }
    }
    wave_sync();
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
    return v;
}

// Nodes of the table of -2 A(r): node i at r = i w, w = sigma / 64.  Row i
// holds the Taylor coefficients in (r - i w) / sigma up to the third, summed
// over the bins whose windows reach any pair the node serves (half a node further
// than 8 sigma).  Relative to a window term at t sigma the remainder over half a node is
// (1/128)^4 / 24 times the fifth Hermite function over t: 1.5e-7 at 6 sigma, 5e-7 at 8;
// float32 window terms by recurrence are 1e-6 (bins of 4 sigma) to 6e-3 (sigma / 40)
// off there.  At sigma / 16 it is 9e-5 and 1.6e-4; the kernel takes as long
// (131,072 points: 239 us whole call, 241 now).  LANES lanes per node: 4 for few terms, where
// the sums over the lanes are most of the work.
template <int LANES>
__global__ void __launch_bounds__(256) smooth_table_kernel(const SmoothArgs a)
{
    const int node = (int)(blockIdx.x * 256 + threadIdx.x) / LANES;
    const int l = threadIdx.x % LANES;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    const double r = (double)node * a.node_w, inv_s = 8.0 / a.w8;
    const double reach = a.w8 + 0.5 * a.node_w;
    if (node < a.nodes) {
        const int b0 = max(0, (int)ceil((r - reach) / a.dr - 0.5));
        const int b1 = min(a.bins - 1, (int)floor((r + reach) / a.dr - 0.5));
        for (int b = b0 + l; b <= b1; b += LANES) {
            const double t = fma((double)b + 0.5, a.dr, -r) * inv_s, t2 = t * t;
            const double e = a.grad_h[b] * exp(-0.5 * t2);
            s0 = fma(e, t, s0);
            s1 = fma(e, t2 - 1.0, s1);
            s2 = fma(e, t * (t2 - 3.0), s2);
            s3 = fma(e, fma(t2, t2 - 6.0, 3.0), s3);
        }
    }
#pragma unroll
    for (int d = LANES / 2; d > 0; d >>= 1) {
        s0 += __shfl_xor(s0, d);
        s1 += __shfl_xor(s1, d);
        s2 += __shfl_xor(s2, d);
        s3 += __shfl_xor(s3, d);
    }
    if (l == 0 && node < a.nodes)
        a.table[node] = make_float4((float)(a.tscale * s0), (float)(a.tscale * s1),
                                    (float)(a.tscale * s2 / 2.0), (float)(a.tscale * s3 / 6.0));
}

// Adjoint flush for the hits of one query: the sum of -2 A(r) d / r, A from the
// table (TABLE) or from its window's terms.
template <int DIM, bool TABLE, int BUF>
__device__ __forceinline__ void flush_bwd(const SmoothArgs& a, const SmoothShared<BUF>& L,
                                          SmoothLds<BUF>& W, const float* G, int nh, int lane,
                                          double& gx, double& gy, double& gz)
{
    wave_sync();
    const float drf = (float)a.dr;
    double ax = 0.0, ay = 0.0, az = 0.0;
    for (int e = lane; e < nh; e += kWave) {
        double dx, dy, dz;
        hit_vector<DIM, BUF>(a, L, W, W.hit[e], dx, dy, dz);
        const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
        if (!(r2 > 0.0)) continue;
        double f;
        if constexpr (TABLE) {
            const double inv_r = inv_sqrt(r2);
            const double r = r2 * inv_r;
            const int i = min((int)fma(r, a.inv_node_w, 0.5), a.nodes - 1);
            const float4 c = a.table[i];
            const float y = (float)(fma(-(double)i, a.node_w, r) * (8.0 / a.w8));
            f = (double)fmaf(fmaf(fmaf(c.w, y, c.z), y, c.y), y, c.x) * inv_r;
        } else {
            const double r = sqrt(r2);
            int b0, b1;
            float u0;
            window(a, r, b0, b1, u0);
            // the window's terms change sign with u: sum them in float64.
            // Consecutive bins' Gaussians by recurrence: with u' = u + dr,
            // e(u') = e(u) p(u) and p(u') = p(u) c, where p(u) =
            // 2^(-k2 (2 u dr + dr^2)) and c = 2^(-2 k2 dr^2); two exp2 per
            // pair instead of one per bin (relative error of a term after
            // the window's ~20 steps: a few 1e-6)
            double A = 0.0;
            const int nb = b1 - b0 + 1;
            float u = u0;
            float e = __builtin_amdgcn_exp2f(-(u * u) * a.k2);
            float p = __builtin_amdgcn_exp2f(-a.k2 * drf * fmaf(2.f, u, drf));
            const float c = a.step2;
            const float* g = G + b0;
#pragma unroll 4
            for (int j = 0; j < nb; ++j) {
                A += (double)(g[j] * u * e);
                e *= p;
                p *= c;
                u += drf;
            }
            f = -2.0 * A / r;
        }
        ax = fma(f, dx, ax);
        ay = fma(f, dy, ay);
        az = fma(f, dz, az);
    }
    gx += wave_sum(ax);
    gy += wave_sum(ay);
    gz += wave_sum(az);
    wave_sync();
}

// TABLE: the adjoint with tabulated A.
template <int DIM, bool BWD, bool TABLE>
__global__ void __launch_bounds__(kBlock) smooth_kernel(const SmoothArgs a)
{
    // the adjoint flushes after every chunk of a query
    constexpr int BUF = BWD ? kSmSlots * kWave : kSmBuf;
    // forward: histogram (float64); adjoint without the table: G (float32)
    extern __shared__ double s_dyn[];
    __shared__ SmoothShared<BUF> L;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uniform(threadIdx.x / kWave);
    SmoothLds<BUF>& W = L.w[wv];
    const PairGeom& G = a.geom;
    if (threadIdx.x < 27) {
        L.off[threadIdx.x] = make_float4(G.off[threadIdx.x][0], G.off[threadIdx.x][1],
                                         G.off[threadIdx.x][2], 0.f);
        for (int c = 0; c < 3; ++c) L.offd[threadIdx.x][c] = a.offd[threadIdx.x][c];
    }
    double* hist = s_dyn;
    float* Gs = reinterpret_cast<float*>(s_dyn);
    for (int b = threadIdx.x; b < (TABLE ? 0 : a.bins); b += kBlock) {
        if (BWD)
            Gs[b] = (float)a.grad_h[b] * a.gscale;
        else
            hist[b] = 0.0;
    }
    __syncthreads();
    const PairIn in{a.cand, a.cand_start, a.cand, a.cand_start};
    const float r2s = G.r2max;
    // work units: each home cell's queries in a.split parts (more units than
    // cells keep enough wavefronts busy when cells are few and full)
    int t0, t1, stride;
    wave_tiles_interleaved<kWavesPerBlock>(G.ncells * a.split, wv, t0, t1, stride);
    int nh = 0;
    auto flush = [&]() {
        flush_fwd<DIM, BUF>(a, L, W, hist, nh, lane);
        nh = 0;
    };
    for (int unit = t0; unit < t1; unit += stride) {
        const int tile = unit / a.split, part = unit - tile * a.split;
        const int qa = in.q_start[tile], qb = in.q_start[tile + 1];
        const int q0 = qa + (int)((long long)(qb - qa) * part / a.split);
        const int q1 = qa + (int)((long long)(qb - qa) * (part + 1) / a.split);
        if (q0 == q1) continue;
        const int C = stencil<DIM>(in, G, tile, lane, W.st);
        for (int c0 = q0; c0 < q1; c0 += kWave) {
            QueryChunk Q;
            Q.load(in, c0, q1 - c0, lane);
            W.q[lane] = Q.q;
            double gx = 0.0, gy = 0.0, gz = 0.0;  // adjoint: lane t holds query t's row
            for (int k0 = 0; k0 < C; k0 += kSmSlots * kWave) {
                SmSlots<DIM, kSmSlots> c;
                c.load(in, G, W.st, L.off, k0, C, lane);
                for (int t = 0; t < Q.n; ++t) {
                    const float qx = lane_off(Q.q.x, t), qy = lane_off(Q.q.y, t);
                    const float qz = DIM == 3 ? lane_off(Q.q.z, t) : 0.f;
                    nh = buffer_query<DIM, kSmSlots, BUF>(c, W, nh, qx, qy, qz, c0 + t, t, r2s, C - k0);
                    if (BWD && nh > 0) {
                        double sx = 0.0, sy = 0.0, sz = 0.0;
                        flush_bwd<DIM, TABLE, BUF>(a, L, W, Gs, nh, lane, sx, sy, sz);
                        nh = 0;
                        if (lane == t) {
                            gx += sx;
                            gy += sy;
                            gz += sz;
                        }
                    } else if (nh >= kSmFlushAt) {
                        flush();
                    }
                }
            }
            if (BWD) {
                if (lane < Q.n) {
                    const int id = Q.my_id();
                    a.grad[3 * (size_t)id] = (float)gx;
                    a.grad[3 * (size_t)id + 1] = (float)gy;
                    a.grad[3 * (size_t)id + 2] = DIM == 3 ? (float)gz : 0.f;
                }
            } else if (nh > 0) {
                flush();  // the query chunk is about to change
            }
            wave_sync();
        }
    }
    if (!BWD) {
        __syncthreads();
        double* out = a.partial + (size_t)blockIdx.x * a.bins;
        for (int b = threadIdx.x; b < a.bins; b += kBlock) out[b] = hist[b];
    }
}

// h[b] += the first stage's sums (level2[row][b]) of the partial histograms.
__global__ void __launch_bounds__(256) smooth_reduce_kernel(const double* __restrict__ level2,
                                                            int rows, int bins,
                                                            double* __restrict__ h)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= bins) return;
    double sum = 0.0;
#pragma unroll 16
    for (int g = 0; g < rows; ++g) sum += level2[(size_t)g * bins + b];
    h[b] += sum;
}

template <int DIM, bool BWD, bool TABLE>
int occupancy_blocks(size_t dyn)
{
    const int per_cu = resident_per_cu(smooth_kernel<DIM, BWD, TABLE>, kBlock, dyn);
    return (device_cus() * per_cu + 7) / 8 * 8;
}

}  // namespace

// Workgroups of a smoothed-RDF launch (the forward's partial histograms are
// sized by it): every workgroup the device holds at once, a multiple of 8.
int smooth_workgroups(bool adjoint, int dim, int bins, bool table)
{
    if (!adjoint) {
        const size_t dyn = sizeof(double) * (size_t)bins;
        return dim == 3 ? occupancy_blocks<3, false, false>(dyn)
                        : occupancy_blocks<2, false, false>(dyn);
    }
    if (table)
        return dim == 3 ? occupancy_blocks<3, true, true>(0) : occupancy_blocks<2, true, true>(0);
    const size_t dyn = sizeof(float) * (size_t)bins;
    return dim == 3 ? occupancy_blocks<3, true, false>(dyn) : occupancy_blocks<2, true, false>(dyn);
}

void launch_smooth_fwd(const SmoothArgs& a, int dim, int blocks, hipStream_t s)
{
    const size_t dyn = sizeof(double) * (size_t)a.bins;
    if (dim == 3)
        hipLaunchKernelGGL((smooth_kernel<3, false, false>), dim3(blocks), dim3(kBlock), dyn, s, a);
    else
        hipLaunchKernelGGL((smooth_kernel<2, false, false>), dim3(blocks), dim3(kBlock), dyn, s, a);
    const int rows = partial_rows(blocks);
    hipLaunchKernelGGL(partial_sum_stage1<double>, dim3((a.bins + 63) / 64, rows), dim3(256), 0, s,
                       a.partial, blocks, a.bins, kPartialRowsPer, a.level2);
    hipLaunchKernelGGL(smooth_reduce_kernel, dim3((a.bins + 255) / 256), dim3(256), 0, s, a.level2,
                       rows, a.bins, a.h);
}

void launch_smooth_bwd(const SmoothArgs& a, int dim, int blocks, hipStream_t s)
{
    if (a.nodes > 0) {
        const int per = 256 / a.node_lanes;
        const dim3 grid((a.nodes + per - 1) / per);
        if (a.node_lanes == 4)
            hipLaunchKernelGGL(smooth_table_kernel<4>, grid, dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL(smooth_table_kernel<16>, grid, dim3(256), 0, s, a);
        if (dim == 3)
            hipLaunchKernelGGL((smooth_kernel<3, true, true>), dim3(blocks), dim3(kBlock), 0, s, a);
        else
            hipLaunchKernelGGL((smooth_kernel<2, true, true>), dim3(blocks), dim3(kBlock), 0, s, a);
        return;
    }
    const size_t dyn = sizeof(float) * (size_t)a.bins;
    if (dim == 3)
        hipLaunchKernelGGL((smooth_kernel<3, true, false>), dim3(blocks), dim3(kBlock), dyn, s, a);
    else
        hipLaunchKernelGGL((smooth_kernel<2, true, false>), dim3(blocks), dim3(kBlock), dyn, s, a);
}

}  // namespace ppa
