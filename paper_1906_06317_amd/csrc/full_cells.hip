// The histogram of full cells: the RDF without a list where a home cell's
// stencil holds more candidates than the fill pass keeps in register slots (a
// cutoff that is large against the points' spacing).
//
// One wavefront takes the queries of one octant of a home cell (a quadrant in
// 2D), or a share of them (PartWalk).  Points near each other share most of their
// candidates, and candidates past the cutoff from the bounding box of the
// wavefront's queries can hit none of them: an octant's box and the cutoff
// cover about 10.5 of the 27 cells' volume, of which a query's ball is 4.2.
// The stencil is streamed cell by cell, tested against the box (cutoff and
// the rounding of the tests, r2prune), and what is left is compacted into an
// LDS stage, from which all the queries take it three register slots at a
// time; the hits' r^2 are compacted again and binned 64 at a time.  In or out
// is decided as in the fill pass without a list, so that a cell's pairs do not depend
// on the route: by r^2 itself where the stencil fits that pass's register slots, by
// the expanded test past them where the host allows it.  Bins come from the
// difference of coordinates.  Bound by vector issue (the tests about half) and, at few wavefronts,
// by the latency of the compactions.  50,021 points, r = 6, 231 points a cell,
// 45 M pairs: 231 us with every query of a cell testing every candidate and
// binning where it was found, 154 us now.  With more bins than fit the LDS the global
// atomics bound either way, and the fill pass is taken.
#include "pair_common.hpp"

namespace ppa {

namespace {

using namespace pair;

constexpr int kR2Cap = 448;      // r^2 buffered per wavefront
constexpr int kStageSlots = 3;
constexpr int kStage = kStageSlots * kWave;
static_assert(2 * kStage <= kR2Cap - kWave, "two queries' hits fit beside a block that waits");

struct FullLds {
    float r2[kR2Cap];
    float4 stage[kStage + kWave];  // the part's queries, then the candidates kept
    StencilLds st;
};

struct FullOut {
    unsigned long long* hist;
    int bins;  // at most kMaxLdsBins
    float r_min, inv_dr;
};

struct FullBins {
    FullLds& W;
    const FullOut O;
    unsigned* hist;  // in LDS
    int lane;
    int nh;          // r^2 waiting

    __device__ __forceinline__ void bin(float r)
    {
        const float t = (r - O.r_min) * O.inv_dr;
        // keeps the four roots of drain() from being issued together with the bins (2 to
        // 6 % of the pass)
        __builtin_amdgcn_sched_barrier(0);
        if (t >= 0.f && t < (float)O.bins) atomicAdd(&hist[min((int)t, O.bins - 1)], 1u);
    }
    // Bins whole blocks of 64 (or with `all` everything); the rest moves up.
    __device__ __forceinline__ void drain(bool all)
    {
        wave_sync();
        int e0 = 0;
        for (; e0 + 4 * kWave <= nh; e0 += 4 * kWave) {  // four reads in flight
            float r2[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) r2[u] = W.r2[e0 + u * kWave + lane];
#pragma unroll
            for (int u = 0; u < 4; ++u) bin(fast_sqrt(r2[u]));
        }
        for (; e0 + kWave <= nh; e0 += kWave) bin(fast_sqrt(W.r2[e0 + lane]));
        float rest = 0.f;
        if (lane < nh - e0) rest = W.r2[e0 + lane];
        if (all) {
            if (lane < nh - e0) bin(fast_sqrt(rest));
            nh = 0;
        } else {
            wave_sync();
            if (lane < nh - e0) W.r2[lane] = rest;
            nh -= e0;
        }
        wave_sync();
    }
    // Hits of query a, and with TWO of b, against the first `count` candidates.
    template <int DIM, int EXCL, bool DOT, bool TWO>
    __device__ __forceinline__ void hits(const Slots<DIM, kStageSlots>& c, const Query& qa,
                                         const Query& qb, float r2max, int count)
    {
        if (nh + (TWO ? 2 : 1) * count > kR2Cap) drain(false);
#pragma unroll
        for (int s = 0; s < kStageSlots; ++s) {
            if (s * kWave >= count) break;  // uniform
            const float ra = dist2<DIM>(c.x[s] - qa.x, c.y[s] - qa.y, c.z[s] - qa.z);
            bool ha = DOT ? c.template hit<true>(s, qa, r2max) : ra < r2max;
            if (EXCL == 2) ha = ha && c.id[s] != qa.id;
            const unsigned long long ma = __ballot(ha);
            if (TWO) {
                const float rb = dist2<DIM>(c.x[s] - qb.x, c.y[s] - qb.y, c.z[s] - qb.z);
                bool hb = DOT ? c.template hit<true>(s, qb, r2max) : rb < r2max;
                if (EXCL == 2) hb = hb && c.id[s] != qb.id;
                const unsigned long long mb = __ballot(hb);
                const int nb = nh + __popcll(ma);
                if (ha) W.r2[nh + (int)lane_prefix(ma)] = ra;
                if (hb) W.r2[nb + (int)lane_prefix(mb)] = rb;
                nh = nb + __popcll(mb);
            } else {
                if (ha) W.r2[nh + (int)lane_prefix(ma)] = ra;
                nh += __popcll(ma);
            }
        }
    }
};

// Every query of the chunk against the first `count` staged candidates.
template <int DIM, int EXCL, bool DOT>
__device__ __forceinline__ void run_stage(FullBins& F, const QueryChunk& Q, float r2max, int count)
{
    wave_sync();
    const int lane = F.lane;
    Slots<DIM, kStageSlots> c;
#pragma unroll
    for (int s = 0; s < kStageSlots; ++s) {
        const int e = s * kWave + lane;
        c.x[s] = c.y[s] = c.z[s] = kFar;
        c.id[s] = -1;
        if (e < count) {
            const float4 v = F.W.stage[e];
            c.x[s] = v.x;
            c.y[s] = v.y;
            c.z[s] = DIM == 3 ? v.z : 0.f;
            c.id[s] = __float_as_int(v.w);
        }
        c.cc[s] = dist2<DIM>(c.x[s], c.y[s], c.z[s]);
    }
    int t = 0;
    for (; t + 1 < Q.n; t += 2)
        F.template hits<DIM, EXCL, DOT, true>(c, Q.template get<DIM>(t, r2max),
                                              Q.template get<DIM>(t + 1, r2max), r2max, count);
    if (t < Q.n) {
        const Query q = Q.template get<DIM>(t, r2max);
        F.template hits<DIM, EXCL, DOT, false>(c, q, q, r2max, count);
    }
}

// Gathers the part's queries first .. first + 63 into the stage: those of the
// home cell's queries [q0, q1) in octant oct, every step-th from the sub-th on.
// Returns how many the part has in all, less `first`.
template <int DIM>
__device__ __forceinline__ int gather_part(const PairIn& in, float4* stage, int q0, int q1, int oct,
                                           int sub, int step, int first, int lane)
{
    wave_sync();
    int seen = 0, taken = 0;  // in the octant, and in the part, so far
    for (int b = q0; b < q1; b += kWave) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (b + lane < q1) v = in.qs[b + lane];
        const int o =
            (v.x >= 0.f ? 1 : 0) | (v.y >= 0.f ? 2 : 0) | (DIM == 3 && v.z >= 0.f ? 4 : 0);
        const bool mine = b + lane < q1 && o == oct;
        const unsigned long long m = __ballot(mine);
        const bool part = mine && (seen + (int)lane_prefix(m)) % step == sub;
        const unsigned long long mp = __ballot(part);
        const int at = taken + (int)lane_prefix(mp) - first;
        if (part && at >= 0 && at < kWave) stage[at] = v;
        seen += __popcll(m);
        taken += __popcll(mp);
    }
    wave_sync();
    return taken - first;
}

// One part of a home cell (octant, share and shares as in gather_part) against
// the cell's stencil in W.st; returns its queries.
template <int DIM, int EXCL, bool DOT>
__device__ __forceinline__ int work_part(const PairIn& in, const PairGeom& G, const float4* s_off,
                                         FullBins& F, int q0, int q1, int oct, int sub, int step)
{
    FullLds& W = F.W;
    const int lane = F.lane;
    const float r2max = G.r2max;
    int all = 0;
    for (int first = 0;; first += kWave) {
        QueryChunk Q;
        Q.n = min(kWave, gather_part<DIM>(in, W.stage, q0, q1, oct, sub, step, first, lane));
        if (Q.n <= 0) break;
        all += Q.n;
        Q.q = W.stage[lane < Q.n ? lane : 0];
        wave_sync();
        // bounding box of the queries
        const float lx = wave_min(Q.q.x), hx = wave_max(Q.q.x);
        const float ly = wave_min(Q.q.y), hy = wave_max(Q.q.y);
        const float lz = DIM == 3 ? wave_min(Q.q.z) : 0.f;
        const float hz = DIM == 3 ? wave_max(Q.q.z) : 0.f;
        int ns = 0;  // candidates staged
        for (int j = 0; j < G.nsten; ++j) {
            const int k0 = uniform(W.st.pre[j]), k1 = uniform(W.st.pre[j + 1]);
            const float4 o = s_off[j];
            const int base = uniform(W.st.base[j]);
            for (int k = k0; k < k1; k += kWave) {
                float4 v = make_float4(kFar, kFar, kFar, 0.f);
                if (k + lane < k1) {
                    v = in.cand[base + k + lane];
                    v.x += o.x;
                    v.y += o.y;
                    v.z = DIM == 3 ? v.z + o.z : 0.f;
                }
                const float dx = fmaxf(fmaxf(v.x - hx, lx - v.x), 0.f);
                const float dy = fmaxf(fmaxf(v.y - hy, ly - v.y), 0.f);
                const float dz = DIM == 3 ? fmaxf(fmaxf(v.z - hz, lz - v.z), 0.f) : 0.f;
                const bool keep = dist2<DIM>(dx, dy, dz) < G.r2prune;
                const unsigned long long m = __ballot(keep);
                if (keep) W.stage[ns + (int)lane_prefix(m)] = v;
                ns += __popcll(m);
                if (ns >= kStage) {
                    run_stage<DIM, EXCL, DOT>(F, Q, r2max, kStage);
                    wave_sync();
                    float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
                    ns -= kStage;
                    if (lane < ns) w = W.stage[kStage + lane];
                    wave_sync();
                    if (lane < ns) W.stage[lane] = w;
                    wave_sync();
                }
            }
        }
        if (ns > 0) run_stage<DIM, EXCL, DOT>(F, Q, r2max, ns);
    }
    return all;
}

// The parts of the home cells: an octant's queries are dealt to shares.  Where
// the cells of an XCD hold about the same (squared counts at most 1.25 of their
// mean's square), every octant has as many shares as make kXcdParts parts (768
// wavefronts of an XCD are resident; 216 cells, 231 points each: 3456 parts in
// all 248 us, 5184 167, 6912 154).  Elsewhere parts are of about equal work, the
// queries times the candidates, taken as the square of a cell's count: droplets
// in a dilute system would keep the few wavefronts that have a part of them long
// after the others ended (20,000 points, three droplets: 1508 us with as many
// shares everywhere, 469 now).  A share keeps kPartQueries queries.  Each
// wavefront counts through its XCD's cells, 64 at a time, and takes every
// stride-th part.
constexpr int kXcdParts = 1024;
constexpr int kPartQueries = 4;

template <int KINDS>
struct PartWalk {
    int cell, c1;        // first of the cells in the lanes, end of the XCD's
    int qb, qn;          // this lane's cell: its first query, its queries,
    int s, incl;         // shares of an octant, and parts up to and with it
    int before;          // parts of the cells before the lanes'
    int k, stride;       // this wavefront's next part
    int alike;           // shares everywhere, or 0 with
    float per_square;    // shares per squared count
    int tile, q0, q1, oct, sub, shares;  // the part

    __device__ __forceinline__ PartWalk(const PairIn& in, const PairGeom& G, int wv, int lane)
    {
        const int xcd = blockIdx.x & 7;
        cell = (int)((long long)xcd * G.ncells / 8);
        c1 = (int)((long long)(xcd + 1) * G.ncells / 8);
        k = (int)(blockIdx.x >> 3) * kWavesPerBlock + wv;
        stride = (int)(gridDim.x >> 3) * kWavesPerBlock;
        before = 0;
        fetch(in, lane);
        float sum = (float)qn, sq = sum * sum;
#pragma unroll 4
        for (int c = cell + kWave + lane; c < c1; c += kWave) {
            const float q = (float)(in.q_start[c + 1] - in.q_start[c]);
            sum += q;
            sq = fmaf(q, q, sq);
        }
        sum = wave_add(sum);
        sq = wave_add(sq);
        const int nc = max(1, c1 - cell);
        const bool even = sq * (float)nc <= 1.25f * sum * sum;
        const int room = (int)(sum / (float)(kPartQueries * KINDS * nc));
        alike = even ? max(1, min(kXcdParts / (KINDS * nc), room)) : 0;
        per_square = (float)(kXcdParts / KINDS) / fmaxf(sq, 1.f);
        deal();
    }
    __device__ __forceinline__ void fetch(const PairIn& in, int lane)
    {
        qb = qn = 0;
        if (cell + lane < c1) {
            qb = in.q_start[cell + lane];
            qn = in.q_start[cell + lane + 1] - qb;
        }
    }
    __device__ __forceinline__ void deal()
    {
        const float q = (float)qn;
        s = alike ? alike : max(1, min((int)(per_square * q * q), qn / (kPartQueries * KINDS)));
        s = qn > 0 ? s : 0;
        incl = wave_incl_scan(KINDS * s);
    }
    // The next part; false at the end.
    __device__ __forceinline__ bool next(const PairIn& in, int lane)
    {
        for (;;) {
            if (k - before < lane_of(incl, kWave - 1)) {
                const int l = __ffsll((long long)__ballot(incl > k - before)) - 1;
                shares = lane_of(s, l);
                tile = uniform(cell + l);
                q0 = lane_of(qb, l);
                q1 = q0 + lane_of(qn, l);
                const int part = k - before - (lane_of(incl, l) - KINDS * shares);
                oct = uniform(part % KINDS);
                sub = uniform(part / KINDS);
                k += stride;
                return true;
            }
            before += lane_of(incl, kWave - 1);
            cell += kWave;
            if (cell >= c1) return false;
            fetch(in, lane);
            deal();
        }
    }
};

// EXCL: 0 keep j == i, 1 points query themselves (each finds its own entry, at
// r = 0, which is taken out of bin 0 at the end), 2 separate query points
// (drop j == i by index).
template <int DIM, int EXCL, bool DOT>
__global__ void __launch_bounds__(kBlock, 6) full_cells_kernel(const PairIn in, const PairGeom G,
                                                               const FullOut O)
{
    extern __shared__ unsigned s_hist[];
    __shared__ float4 s_off[27];
    __shared__ FullLds s_w[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uniform(threadIdx.x / kWave);
    FullLds& W = s_w[wv];
    if (threadIdx.x < 27)
        s_off[threadIdx.x] = make_float4(G.off[threadIdx.x][0], G.off[threadIdx.x][1],
                                         G.off[threadIdx.x][2], 0.f);
    for (int b = threadIdx.x; b < O.bins; b += kBlock) s_hist[b] = 0u;
    __syncthreads();
    FullBins F{W, O, s_hist, lane, 0};
    int selfs = 0;
    PartWalk<DIM == 3 ? 8 : 4> P(in, G, wv, lane);
    while (P.next(in, lane)) {
        const int C = stencil<DIM>(in, G, P.tile, lane, W.st);
        if (DOT && C > kFillSlots * kWave)
            selfs += work_part<DIM, EXCL, true>(in, G, s_off, F, P.q0, P.q1, P.oct, P.sub,
                                                P.shares);
        else
            selfs += work_part<DIM, EXCL, false>(in, G, s_off, F, P.q0, P.q1, P.oct, P.sub,
                                                 P.shares);
    }
    F.drain(true);
    if (EXCL == 1 && selfs > 0 && O.r_min <= 0.f && lane == 0)
        atomicSub(&s_hist[0], (unsigned)selfs);
    __syncthreads();
    for (int b = threadIdx.x; b < O.bins; b += kBlock) {
        const unsigned v = s_hist[b];
        if (v) atomicAdd(&O.hist[b], (unsigned long long)v);
    }
}

template <int DIM, int EXCL, bool DOT>
void launch_full_t(const PairIn& in, const PairGeom& g, const FullOut& o, int64_t nq, hipStream_t s)
{
    const size_t lds = sizeof(unsigned) * (size_t)o.bins;
    const auto k = full_cells_kernel<DIM, EXCL, DOT>;
    const long long more = nq / kPartQueries;  // parts past one an octant, at most
    const long long parts = (long long)g.ncells * (DIM == 3 ? 8 : 4) +
                            (more < 8 * kXcdParts ? more : 8 * kXcdParts);
    hipLaunchKernelGGL(k, dim3(resident_blocks(k, lds, parts)), dim3(kBlock), lds, s, in, g, o);
}

}  // namespace

void launch_full_cells(const PairArgs& a, int dim, int excl, int64_t nq, hipStream_t s)
{
    const PairIn in{a.cand, a.cand_start, a.qsorted, a.q_start};
    const FullOut o{a.hist, a.bins, a.r_min, a.inv_dr};
#define PPA_FULL(D, E)                                         \
    do {                                                       \
        if (a.geom.dot) launch_full_t<D, E, true>(in, a.geom, o, nq, s); \
        else launch_full_t<D, E, false>(in, a.geom, o, nq, s);     \
    } while (0)
    if (dim == 3) {
        if (excl == 1) PPA_FULL(3, 1); else if (excl == 2) PPA_FULL(3, 2); else PPA_FULL(3, 0);
    } else {
        if (excl == 1) PPA_FULL(2, 1); else if (excl == 2) PPA_FULL(2, 2); else PPA_FULL(2, 0);
    }
#undef PPA_FULL
}

}  // namespace ppa
