// Rows of a NeighborList ordered by neighbour index (the paper's promise of
// sorted neighbour order in the Python API, "Implementation"; the analyses do
// not need it, so it is an option of the query).
//
// One wavefront per row, rows dealt to wavefronts in turn.  A row of at
// most kSortLds entries is staged in LDS (indices and distances); each
// entry's place is the number of entries of the row with a smaller index
// (indices are distinct within a row), and the wavefront writes the row back
// in that order.  Longer rows are sorted in place in global memory by a
// bitonic network whose comparators all put the smaller key first, so the
// missing entries of the padded power-of-two length (taken as +infinity)
// never move into the row.
//
// A row that the list could hold only in part (its capacity exceeded) stays in
// the unsorted order, stencil cell by stencil cell and by index within one, like
// the list it is the end of.  The cells of a query with sorted rows are not
// ordered by index, so the fill pass leaves that one row in the order of arrival: it is
// written again here.
#include "pair_common.hpp"

namespace ppa {

namespace {

using namespace pair;

constexpr int kSortBlock = 256;
constexpr int kSortWaves = kSortBlock / kWave;
constexpr int kSortLds = 256;  // entries a wavefront stages in LDS

// Orders a, b (positions in the row, b > a) so the smaller index comes first.
__device__ __forceinline__ void compare_swap(int32_t* idx, float* dist, long long a, long long b)
{
    const int ka = idx[a], kb = idx[b];
    if (kb < ka) {
        idx[a] = kb;
        idx[b] = ka;
        if (dist) {
            const float da = dist[a];
            dist[a] = dist[b];
            dist[b] = da;
        }
    }
}

// In-place bitonic sort of row [e0, e0 + L) in global memory.  For each
// merge size k: first every element of the lower half of a block meets its
// mirror image in the upper half, then half-cleaners at distances k/4 ... 1.
// Partners past the end of the row are +infinity and stay where they are.
__device__ void bitonic_row(int32_t* idx, float* dist, long long e0, long long L, int lane)
{
    int lp = 0;  // P = 2^lp >= L
    while ((1LL << lp) < L) ++lp;
    const long long pairs = 1LL << (lp - 1);
    int32_t* ri = idx + e0;
    float* rd = dist ? dist + e0 : nullptr;
    for (int lk = 1; lk <= lp; ++lk) {  // merge size k = 2^lk
        const long long k = 1LL << lk, hmask = (k >> 1) - 1;
        for (long long t = lane; t < pairs; t += kWave) {
            const long long blk = (t >> (lk - 1)) << lk;
            const long long a = blk + (t & hmask);
            const long long b = blk + (k - 1 - (t & hmask));
            if (b < L) compare_swap(ri, rd, a, b);
        }
        // stores of this step are read by other lanes in the next one
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
        for (int lj = lk - 2; lj >= 0; --lj) {  // half-cleaners at distance 2^lj
            const long long j = 1LL << lj;
            for (long long t = lane; t < pairs; t += kWave) {
                const long long a = ((t >> lj) << (lj + 1)) + (t & (j - 1));
                const long long b = a + j;
                if (b < L) compare_swap(ri, rd, a, b);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// The query of a single frame's rows: its points and geometry, and the queries'
// home cells.
struct RowSource {
    PairIn in;
    PairGeom geom;
    const int* home;
    int excl;
};

// Writes the hits of query `row` to [e0, capacity) in the unsorted order, by the
// fill pass's test and distance; each candidate's place in its cell is the number of hits
// there with a smaller index.
template <int DIM>
__device__ void cut_row(const RowSource& Q, StencilLds& S, int row, long long e0,
                        int64_t capacity, int32_t* idx, float* dist, int lane)
{
    const PairGeom& G = Q.geom;
    const int home = uniform(Q.home[row]);
    Query q = make_query<DIM>(0.f, 0.f, 0.f, row, G.r2max);
    for (int b = Q.in.q_start[home], e = Q.in.q_start[home + 1]; b < e; b += kWave) {
        const float4 v = Q.in.qs[b + lane < e ? b + lane : e - 1];
        const unsigned long long m = __ballot(__float_as_int(v.w) == row);
        if (m) {
            const int l = __ffsll((long long)m) - 1;
            q = make_query<DIM>(lane_off(v.x, l), lane_off(v.y, l), lane_off(v.z, l), row, G.r2max);
            break;
        }
    }
    (void)stencil<DIM>(Q.in, G, home, lane, S);
    long long w = e0;
    for (int j = 0; j < G.nsten && w < capacity; ++j) {
        const int k1 = uniform(S.pre[j + 1]), base = uniform(S.base[j]);
        auto test = [&](int k, Slots<DIM, 1>& c) {
            const float4 v = Q.in.cand[base + k];
            c.x[0] = v.x + G.off[j][0];
            c.y[0] = v.y + G.off[j][1];
            c.z[0] = DIM == 3 ? v.z + G.off[j][2] : 0.f;
            c.id[0] = __float_as_int(v.w);
            c.cc[0] = dist2<DIM>(c.x[0], c.y[0], c.z[0]);
            const bool h = G.dot ? c.template hit<true>(0, q, G.r2max)
                                 : c.template hit<false>(0, q, G.r2max);
            return h && !(Q.excl != 0 && c.id[0] == row);
        };
        int found = 0;
        for (int k0 = uniform(S.pre[j]); k0 < k1; k0 += kWave) {
            Slots<DIM, 1> c;
            const bool h = test(min(k0 + lane, k1 - 1), c) && k0 + lane < k1;
            int before = 0;
            for (int k = uniform(S.pre[j]); k < k1; ++k) {
                Slots<DIM, 1> o;
                if (test(k, o) && o.id[0] < c.id[0]) ++before;
            }
            if (h && w + before < capacity) {
                idx[w + before] = c.id[0];
                if (dist)
                    dist[w + before] = fast_sqrt(
                        dist2<DIM>(c.x[0] - q.x, c.y[0] - q.y, c.z[0] - q.z));
            }
            found += __popcll(__ballot(h));
        }
        w += found;
    }
    wave_sync();
}

// DIM: of the query whose rows these are, with `source`; 0 where the cells are ordered.
template <int DIM>
__global__ void __launch_bounds__(kSortBlock) sort_rows_kernel(const int64_t* __restrict__ offsets,
                                                               int64_t nq, int32_t* idx,
                                                               float* dist, int64_t capacity,
                                                               const RowSource source)
{
    __shared__ StencilLds s_st[DIM > 0 ? kSortWaves : 1];
    __shared__ alignas(16) int s_key[kSortWaves][kSortLds];
    __shared__ float s_val[kSortWaves][kSortLds];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x / kWave;
    int* key = s_key[wv];
    float* val = s_val[wv];
    const long long nwaves = (long long)gridDim.x * kSortWaves;
    for (long long row = (long long)blockIdx.x * kSortWaves + wv; row < nq; row += nwaves) {
        const long long e0 = offsets[row], e1 = offsets[row + 1];
        // rows the list could not hold (capacity exceeded) stay unsorted
        if (e0 < 0 || e1 < e0 || e1 > capacity) continue;
        const long long L = e1 - e0;
        if (L < 2) continue;
        if (L > kSortLds) {
            bitonic_row(idx, dist, e0, L, lane);
            continue;
        }
        const int n = (int)L;
        const int n4 = (n + 3) & ~3;
        for (int e = lane; e < n4; e += kWave) {
            key[e] = e < n ? idx[e0 + e] : 0x7fffffff;  // padding sorts last
            if (dist && e < n) val[e] = dist[e0 + e];
        }
        wave_sync();
        for (int e = lane; e < n; e += kWave) {
            const int mine = key[e];
            int r = 0;
            for (int u = 0; u < n4; u += 4) {
                const int4 v = *reinterpret_cast<const int4*>(&key[u]);
                r += (v.x < mine) + (v.y < mine) + (v.z < mine) + (v.w < mine);
            }
            idx[e0 + r] = mine;
            if (dist) dist[e0 + r] = val[e];
        }
        wave_sync();  // the next row reuses the buffers
    }
    if constexpr (DIM > 0) {
        // the last row that begins before the capacity, if it is cut off, by the wavefront
        // that met it
        if (offsets[nq] <= capacity || capacity <= 0) return;
        long long lo = 0, hi = nq;  // offsets[lo] < capacity < offsets[hi], if there is such a row
        while (hi - lo > 1) {
            const long long mid = (lo + hi) / 2;
            if (offsets[mid] < capacity)
                lo = mid;
            else
                hi = mid;
        }
        const long long me = (long long)blockIdx.x * kSortWaves + wv;
        if (lo % nwaves == me && offsets[lo] >= 0 && offsets[lo + 1] > capacity)
            cut_row<DIM>(source, s_st[wv], (int)lo, offsets[lo], capacity, idx, dist, lane);
    }
}

}  // namespace

static int sort_blocks(int64_t nq)
{
    const long long blocks = (nq + kSortWaves - 1) / kSortWaves, cap = 16LL * device_cus();
    return (int)(blocks < cap ? blocks : cap);
}

void launch_sort_rows(const int64_t* offsets, int64_t nq, int32_t* idx, float* dist,
                      int64_t capacity, hipStream_t s)
{
    if (nq <= 0 || !idx) return;
    hipLaunchKernelGGL(sort_rows_kernel<0>, dim3(sort_blocks(nq)), dim3(kSortBlock), 0, s, offsets,
                       nq, idx, dist, capacity, RowSource{});
}

void launch_sort_query_rows(const PairArgs& a, const int* home, int64_t nq, int dim, int excl,
                            hipStream_t s)
{
    if (nq <= 0 || !a.point_idx) return;
    const RowSource q{PairIn{a.cand, a.cand_start, a.qsorted, a.q_start}, a.geom, home, excl};
    const auto k = dim == 3 ? sort_rows_kernel<3> : sort_rows_kernel<2>;
    hipLaunchKernelGGL(k, dim3(sort_blocks(nq)), dim3(kSortBlock), 0, s, a.offsets, nq,
                       a.point_idx, a.dist, a.capacity, q);
}

}  // namespace ppa
