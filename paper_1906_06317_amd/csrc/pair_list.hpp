// Ball query over the cell list, with the RDF histogram binned in the same
// pass (the paper's neighbor query with a distance cutoff and the density
// module's RDF, "General Utilities" and "Analysis Modules": finding pairs
// inside the analysis instead of materializing them first is the design the
// paper credits with a 2x speed-up).
//
// Work decomposition (one wavefront per home cell):
//   * the home cells of an XCD are contiguous, and its wavefronts take them in
//     turn (lists of long cells: the last quarter from a queue), so the cells
//     in flight are neighbours and its L2 sees their stencils overlap;
//   * for a home cell, the 27 (2D: 9) stencil cells are gathered into NS
//     64-wide slots held in registers, each candidate shifted by its stencil
//     offset so it is relative to the home cell's centre; the code for each
//     slot count NS is unrolled separately, so the slot loop has no branches;
//   * the home cell's query points are prefetched 64 at a time into lanes
//     and read into scalar registers one by one; each is tested against
//     every slot with one ballot per slot.
// The in/out test of a candidate c against query q is either the plain
// |c - q|^2 < r_max^2 or, when the host has bounded its rounding error well
// inside the parity band, the expanded |c|^2 - 2 c.q < r_max^2 - |q|^2 (three
// FMAs).  The count pass keeps -2c and |c|^2 in its slots and reads each
// query, with its r_max^2 - |q|^2, from a per-wavefront LDS row by one
// broadcast load, so the tests take all operands from vector registers; two
// queries go at a time.  The fill pass keeps c and forms -2q per query; the
// products (-2c).q and c.(-2q) are equal and exact inside the FMA, so both
// passes evaluate the same value and agree pair by pair.  Every reported
// distance and bin is recomputed from the difference c - q.
// The NeighborList takes two passes so rows land in query order without
// atomics: count_kernel writes row lengths, a scan turns them into CSR
// offsets, and fill_kernel compacts hits with ballot + mbcnt into a small
// per-wavefront LDS list of whole rows, flushed densely: the distance, the
// histogram bin and coalesced stores for 64 hits per instruction.  Since the
// count pass fixed every row's length, the fill pass tests two queries
// against the same candidate registers at once and places the second row
// right after the first before either is found; the two independent chains
// interleave.  The RDF alone (no list) needs only the fill pass, or over full
// cells one of its own.  Stencils with more candidates than the register slots
// hold are processed in chunks, writing directly.
#pragma once

#include "pair_common.hpp"

namespace ppa {

namespace {

using namespace pair;

constexpr int kHitCap = 320;  // hits buffered per wavefront between flushes
constexpr int kRows = 64;     // rows buffered per wavefront (in a batch, kBatchRows)
static_assert(kFillSlots * kWave <= kCandCap, "a whole stencil fits the r^2 buffer");
constexpr int kMaxBatchLdsBins = 1024;  // per-wavefront histograms of a batch up to this size

// ---------------------------------------------------------------------------
// Pass 1: row lengths.
// ---------------------------------------------------------------------------
// Row lengths of the tile's queries, expanded test: candidates as -2c and
// |c|^2, each query's coordinates and r_max^2 - |q|^2 read from its lane
// (four readlanes), then three FMAs and a compare per slot.
template <int DIM, int EXCL, int NS>
__device__ __forceinline__ void count_tile_dot(const PairIn& in, const GeomView& G,
                                               const StencilLds& S, const float4* off, int C,
                                               int q0, int q1, int lane, float4* qrow,
                                               int32_t* __restrict__ counts)
{
    DotSlots<DIM, NS> c;
    c.load(in, G.nsten, S, off, 0, C, lane);
    for (int c0 = q0; c0 < q1; c0 += kWave) {
        DotChunk Q;
        Q.template load<DIM>(in, c0, q1 - c0, lane, G.r2max, qrow);
        int cnt_v = 0;
        // two queries at a time: two independent test chains interleave
        int t = 0;
        for (; t + 1 < Q.n; t += 2) {
            const DQuery qa = Q.get(t);
            const DQuery qb = Q.get(t + 1);
            int na = 0, nb = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                bool ha = c.hit(s, qa.x, qa.y, qa.z, qa.thr);
                bool hb = c.hit(s, qb.x, qb.y, qb.z, qb.thr);
                if (EXCL == 2) {
                    ha = ha && c.id[s] != qa.id;
                    hb = hb && c.id[s] != qb.id;
                }
                na += __popcll(__ballot(ha));
                nb += __popcll(__ballot(hb));
            }
            // a point querying itself always finds its own entry, at r = 0
            if (EXCL == 1) {
                na -= 1;
                nb -= 1;
            }
            cnt_v = with_lane(cnt_v, t, na);
            cnt_v = with_lane(cnt_v, t + 1, nb);
        }
        if (t < Q.n) {
            const DQuery q = Q.get(t);
            int n = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                bool h = c.hit(s, q.x, q.y, q.z, q.thr);
                if (EXCL == 2) h = h && c.id[s] != q.id;
                n += __popcll(__ballot(h));
            }
            if (EXCL == 1) n -= 1;
            cnt_v = with_lane(cnt_v, t, n);
        }
        if (lane < Q.n) counts[Q.my_id()] = cnt_v;
    }
}

// The same with the plain test |c - q|^2 < r_max^2 (when the host could not
// bound the expanded test's rounding inside the parity band).
template <int DIM, int EXCL, int NS>
__device__ __forceinline__ void count_tile_plain(const PairIn& in, const GeomView& G,
                                                 const StencilLds& S, const float4* off, int C,
                                                 int q0, int q1, int lane,
                                                 int32_t* __restrict__ counts)
{
    Slots<DIM, NS> c;
    c.load(in, G.nsten, S, off, 0, C, lane);
    const float r2max = G.r2max;
    for (int c0 = q0; c0 < q1; c0 += kWave) {
        QueryChunk Q;
        Q.load(in, c0, q1 - c0, lane);
        int cnt_v = 0;
        for (int t = 0; t < Q.n; ++t) {
            const Query q = Q.get<DIM>(t, r2max);
            int n = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                bool h = c.template hit<false>(s, q, r2max);
                if (EXCL == 2) h = h && c.id[s] != q.id;
                n += __popcll(__ballot(h));
            }
            if (EXCL == 1) n -= 1;
            cnt_v = with_lane(cnt_v, t, n);
        }
        if (lane < Q.n) counts[Q.my_id()] = cnt_v;
    }
}

// Stencils too large for the register slots: candidate chunks of
// kChunkSlots slots, each loaded once per 64 queries.
template <int DIM, int EXCL>
__device__ __forceinline__ void count_chunked(const PairIn& in, const GeomView& G,
                                              const StencilLds& S, const float4* off, int C,
                                              int q0, int q1, int lane,
                                              int32_t* __restrict__ counts)
{
    const float r2max = G.r2max;
    for (int c0 = q0; c0 < q1; c0 += kWave) {
        QueryChunk Q;
        Q.load(in, c0, q1 - c0, lane);
        int cnt_v = EXCL == 1 ? -1 : 0;
        for (int k0 = 0; k0 < C; k0 += kChunkSlots * kWave) {
            Slots<DIM, kChunkSlots> c;
            c.load(in, G.nsten, S, off, k0, C, lane);
            for (int t = 0; t < Q.n; ++t) {
                const Query q = Q.get<DIM>(t, r2max);
                int n = 0;
#pragma unroll
                for (int s = 0; s < kChunkSlots; ++s) {
                    bool h = G.dot ? c.template hit<true>(s, q, r2max)
                                   : c.template hit<false>(s, q, r2max);
                    if (EXCL == 2) h = h && c.id[s] != q.id;
                    n += __popcll(__ballot(h));
                }
                cnt_v += lane == t ? n : 0;
            }
        }
        if (lane < Q.n) counts[Q.my_id()] = cnt_v;
    }
}

// Row lengths of one home cell: the slot count picks the unrolled code.
template <int DIM, int EXCL>
__device__ __forceinline__ void count_cell(const PairIn& in, const GeomView& V,
                                           const StencilLds& S, const float4* off, int C, int q0,
                                           int q1, int lane, float4* qrow,
                                           int32_t* __restrict__ counts)
{
    const int ns = (C + kWave - 1) / kWave;
    if (V.dot) {
        switch (ns) {
#define PPA_CASE(N) \
    case N: count_tile_dot<DIM, EXCL, N>(in, V, S, off, C, q0, q1, lane, qrow, counts); return;
            PPA_CASE(0) PPA_CASE(1) PPA_CASE(2) PPA_CASE(3) PPA_CASE(4) PPA_CASE(5) PPA_CASE(6)
            PPA_CASE(7) PPA_CASE(8) PPA_CASE(9) PPA_CASE(10) PPA_CASE(11) PPA_CASE(12)
#undef PPA_CASE
        default: break;
        }
    } else {
        switch (ns) {
#define PPA_CASE(N) \
    case N: count_tile_plain<DIM, EXCL, N>(in, V, S, off, C, q0, q1, lane, counts); return;
            PPA_CASE(0) PPA_CASE(1) PPA_CASE(2) PPA_CASE(3) PPA_CASE(4) PPA_CASE(5) PPA_CASE(6)
            PPA_CASE(7) PPA_CASE(8) PPA_CASE(9) PPA_CASE(10) PPA_CASE(11) PPA_CASE(12)
#undef PPA_CASE
        default: break;
        }
    }
    count_chunked<DIM, EXCL>(in, V, S, off, C, q0, q1, lane, counts);
}

// ---------------------------------------------------------------------------
// Pass 2 (or the only pass for the histogram alone): hits -> list / bins.
// ---------------------------------------------------------------------------
struct FillOut {
    const int64_t* __restrict__ offsets;  // CSR row pointer (NL)
    int32_t* point_idx;
    float* dist;
    int64_t capacity;
    unsigned* status;
    unsigned long long* hist;
    int bins;
    float r_min;
    float inv_dr;
};

// Per-wavefront LDS of the fill pass.  With a list, a hit keeps the
// candidate's coordinates (its exact distance is recomputed at the flush)
// and rows are whole; for the histogram alone, a hit keeps only its exact
// r^2 from the difference form.
template <bool NL, int ROWS = kRows>
struct FillLds;

template <int ROWS>
struct FillLds<true, ROWS> {
    float4 hit[kHitCap];               // candidate xyz relative to the home centre, index bits
    float4 rq[ROWS];                   // each non-empty row's query xyz, index bits
    long long base[ROWS];              // offsets[q] - first buffered hit of the row
    unsigned long long starts[kHitCap / 64];  // bit e: a non-empty row starts at hit e
    StencilLds st;
};

template <int ROWS>
struct FillLds<false, ROWS> {
    float r2[kCandCap];
    StencilLds st;
};

// Per-wavefront state of the fill pass.
template <int DIM, int EXCL, bool NL, bool HIST, int ROWS = kRows>
struct Filler {
    FillLds<NL, ROWS>& W;
    const FillOut O;
    unsigned* hist_lds;  // NULL: bin straight into ghist
    unsigned long long* ghist;  // the histogram in global memory (the frame's, in a batch)
    int id_base;  // subtracted from point indices written to the list (frame-local indices)
    int lane;
    int nh;     // hits buffered
    int nrows;  // rows buffered
    int selfs;  // own entries binned by the histogram-only path (all at r = 0)
    bool over;

    __device__ Filler(FillLds<NL, ROWS>& w, const FillOut& o, unsigned* h, int l)
        : W(w), O(o), hist_lds(h), ghist(o.hist), id_base(0), lane(l), nh(0), nrows(0), selfs(0),
          over(false)
    {
    }

    __device__ __forceinline__ void bin_at(float t)
    {
        const int b = min((int)t, O.bins - 1);
        if (hist_lds)
            atomicAdd(&hist_lds[b], 1u);
        else
            atomicAdd(&ghist[b], 1ull);
    }
    __device__ __forceinline__ void bin(float r)
    {
        if (O.r_min == 0.f) {
            // r >= 0, and r - 0 is r: the same t without the subtraction or
            // the lower test
            const float t = r * O.inv_dr;
            if (t < (float)O.bins) bin_at(t);
        } else {
            const float t = (r - O.r_min) * O.inv_dr;
            if (t >= 0.f && t < (float)O.bins) bin_at(t);
        }
    }
    __device__ __forceinline__ void emit(long long dst, int id, float r)
    {
        if (dst < O.capacity) {
            // the list is written once and read by a later kernel: stream it
            // past the caches, which keep the stencil cells
            __builtin_nontemporal_store(id - id_base, &O.point_idx[dst]);
            if (O.dist) __builtin_nontemporal_store(r, &O.dist[dst]);
        } else {
            over = true;
        }
    }
    // Records a buffered row starting at position rs: query t of the chunk
    // (its lane holds the point and its row offset rb_v) writes the record
    // and the row's start bit.
    __device__ __forceinline__ void add_row(const QueryChunk& Q, long long rb_v, int t, int rs)
    {
        if constexpr (NL) {
            if (lane == t) {
                W.rq[nrows] = Q.q;
                W.base[nrows] = rb_v - rs;
                // the two rows of a pair may share a word: different lanes
                atomicOr(&W.starts[rs >> 6], 1ull << (rs & 63));
            }
            ++nrows;
        }
    }
    // Emits every buffered hit: exact distance, list store and histogram bin.
    // The row of hit e is the number of row starts at or before e, minus one.
    __device__ __forceinline__ void flush()
    {
        wave_sync();
        if constexpr (NL) {
            // every block's row starts by one read: lane b holds block b's word
            unsigned long long sw = 0ull;
            if (lane < kHitCap / 64) sw = W.starts[lane];
            int before = 0;  // row starts in earlier 64-hit blocks
            for (int e0 = 0; e0 < nh; e0 += kWave) {
                const unsigned long long bm = (unsigned long long)lane_of64((long long)sw, e0 >> 6);
                const int e = e0 + lane;
                // starts at hits e0 .. e: those at bits 1 .. lane counted by
                // the mbcnt of bm >> 1, plus bit 0
                const int r = lane_slot(bm >> 1, before + (int)(bm & 1ull) - 1);
                before += __popcll(bm);
                if (e < nh) {
                    // the three reads depend only on e and r: issue them together
                    const float4 h = W.hit[e];
                    const float4 q = W.rq[r];
                    const long long b = W.base[r];
                    // keep the index with the rest of the record's read (one
                    // 16-byte read, not a second one in the store branch)
                    int id = __float_as_int(h.w);
                    asm volatile("" : "+v"(id));
                    const float d = fast_sqrt(dist2<DIM>(h.x - q.x, h.y - q.y, h.z - q.z));
                    emit(b + e, id, d);
                    if (HIST) bin(d);
                }
            }
            if (lane < kHitCap / 64) W.starts[lane] = 0ull;
        } else {
            for (int e = lane; e < nh; e += kWave) bin(fast_sqrt(W.r2[e]));
        }
        nh = 0;
        nrows = 0;
        wave_sync();
    }

    // Buffers the hits of query q against NS slots.  For a point querying
    // itself, its own entry is lane `self` of slot 0 (the home cell comes
    // first in the stencil and lists its points in query order); BY_ID drops
    // the entry with the query's index instead (separate query points, or a
    // home cell too full for the lane rule).
    template <int NS, bool DOT, bool BY_ID>
    __device__ __forceinline__ void buffer_hits(const Slots<DIM, NS>& c, const Query& q,
                                                float r2max, int self)
    {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if constexpr (NL) {
                bool h = c.template hit<DOT>(s, q, r2max);
                if (BY_ID) h = h && c.id[s] != q.id;
                if (!BY_ID && EXCL == 1 && s == 0) h = h && lane != self;
                const unsigned long long m = __ballot(h);
                if (h) {
                    float4* dst = &W.hit[nh];
                    dst[lane_prefix(m)] =
                        make_float4(c.x[s], c.y[s], c.z[s], __int_as_float(c.id[s]));
                }
                nh += __popcll(m);
            } else {
                const float r2 = dist2<DIM>(c.x[s] - q.x, c.y[s] - q.y, c.z[s] - q.z);
                bool h = r2 < r2max;
                if (EXCL == 2) h = h && c.id[s] != q.id;
                const unsigned long long m = __ballot(h);
                if (h) W.r2[nh + (int)lane_prefix(m)] = r2;
                nh += __popcll(m);
            }
        }
        // the histogram-only path keeps a point's own entry (r = 0) and
        // removes it from bin 0 at the end
        if (!NL && EXCL == 1) ++selfs;
    }
    // Buffers the hits of two queries at once: a's row (its length known
    // from the count pass) at wa, b's at wb, right after it.  The two in/out
    // chains share the candidate registers and are independent, so their
    // instructions interleave.
    template <int NS, bool DOT, bool BY_ID>
    __device__ __forceinline__ void buffer_pair(const Slots<DIM, NS>& c, const Query& qa,
                                                const Query& qb, float r2max, int self_a,
                                                int self_b, int wa, int wb)
    {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            bool ha = c.template hit<DOT>(s, qa, r2max);
            bool hb = c.template hit<DOT>(s, qb, r2max);
            if (BY_ID) {
                ha = ha && c.id[s] != qa.id;
                hb = hb && c.id[s] != qb.id;
            }
            if (!BY_ID && EXCL == 1 && s == 0) {
                ha = ha && lane != self_a;
                hb = hb && lane != self_b;
            }
            const unsigned long long ma = __ballot(ha);
            const unsigned long long mb = __ballot(hb);
            const float4 v = make_float4(c.x[s], c.y[s], c.z[s], __int_as_float(c.id[s]));
            if (ha) W.hit[wa + (int)lane_prefix(ma)] = v;
            if (hb) W.hit[wb + (int)lane_prefix(mb)] = v;
            wa += __popcll(ma);
            wb += __popcll(mb);
        }
    }
    // Writes the hits of query q against NS slots straight to the outputs,
    // at rbase + w onwards.
    template <int NS, bool DOT>
    __device__ __forceinline__ void direct_hits(const Slots<DIM, NS>& c, const Query& q,
                                                float r2max, long long rbase, int& w)
    {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            bool h = c.template hit<DOT>(s, q, r2max);
            if (EXCL != 0) h = h && c.id[s] != q.id;
            const unsigned long long m = __ballot(h);
            if (h) {
                const float d = fast_sqrt(dist2<DIM>(c.x[s] - q.x, c.y[s] - q.y, c.z[s] - q.z));
                if (NL) emit(rbase + w + (int)lane_prefix(m), c.id[s], d);
                if (HIST) bin(d);
            }
            w += __popcll(m);
        }
    }
};

// Queries [q0, q1) of the home cell whose first query is qc.
template <int DIM, int EXCL, bool NL, bool HIST, int NS, int ROWS>
__device__ __forceinline__ void fill_tile(const PairIn& in, const GeomView& G, const StencilLds& S,
                                          const float4* off, int C, int qc, int q0, int q1,
                                          Filler<DIM, EXCL, NL, HIST, ROWS>& F)
{
    const int lane = F.lane;
    Slots<DIM, NS> c;
    c.load(in, G.nsten, S, off, 0, C, lane);
    const float r2max = G.r2max;
    for (int c0 = q0; c0 < q1; c0 += kWave) {
        QueryChunk Q;
        Q.load(in, c0, q1 - c0, lane);
        long long rb_v = 0;
        int rl_v = 0;
        if (NL && lane < Q.n) {
            rb_v = F.O.offsets[Q.my_id()];
            rl_v = (int)(F.O.offsets[Q.my_id() + 1] - rb_v);
        }
        for (int t = 0; t < Q.n; ++t) {
            // position of the query's own entry in slot 0 (home cell first)
            const int self = (c0 - qc) + t < kWave ? (c0 - qc) + t : -1;
            if constexpr (NL) {
                const int need = lane_of(rl_v, t);  // the row, from the count pass
                if (need > kHitCap) {
                    int w = 0;
                    const long long rbase = lane_of64(rb_v, t);
                    if (G.dot)
                        F.template direct_hits<NS, true>(c, Q.get<DIM>(t, r2max), r2max, rbase, w);
                    else
                        F.template direct_hits<NS, false>(c, Q.get<DIM>(t, r2max), r2max, rbase, w);
                    continue;
                }
                // two rows at once when both fit the buffer
                const int need_b = t + 1 < Q.n ? lane_of(rl_v, t + 1) : kHitCap + 1;
                if (need + need_b <= kHitCap) {
                    if (F.nh + need + need_b > kHitCap || F.nrows + 2 > ROWS) F.flush();
                    const int rsa = F.nh;
                    const int rsb = rsa + need;
                    const int self_b = (c0 - qc) + t + 1 < kWave ? (c0 - qc) + t + 1 : -1;
                    const bool by_id = EXCL == 2 || (EXCL == 1 && self_b < 0);
                    const Query qa = Q.get<DIM>(t, r2max);
                    const Query qb = Q.get<DIM>(t + 1, r2max);
                    if (G.dot) {
                        if (by_id)
                            F.template buffer_pair<NS, true, true>(c, qa, qb, r2max, self, self_b,
                                                                   rsa, rsb);
                        else
                            F.template buffer_pair<NS, true, false>(c, qa, qb, r2max, self, self_b,
                                                                    rsa, rsb);
                    } else {
                        if (by_id)
                            F.template buffer_pair<NS, false, true>(c, qa, qb, r2max, self,
                                                                    self_b, rsa, rsb);
                        else
                            F.template buffer_pair<NS, false, false>(c, qa, qb, r2max, self,
                                                                     self_b, rsa, rsb);
                    }
                    if (need > 0) F.add_row(Q, rb_v, t, rsa);
                    if (need_b > 0) F.add_row(Q, rb_v, t + 1, rsb);
                    F.nh = rsb + need_b;
                    ++t;
                    continue;
                }
                if (F.nh + need > kHitCap || F.nrows == ROWS) F.flush();
            } else {
                // the histogram alone: at most every candidate
                if (F.nh + C > kCandCap) F.flush();
            }
            const int rs = F.nh;
            const bool by_id = EXCL == 2 || (EXCL == 1 && self < 0);
            const Query q = Q.get<DIM>(t, r2max);
            if (NL && G.dot) {
                if (by_id)
                    F.template buffer_hits<NS, true, true>(c, q, r2max, self);
                else
                    F.template buffer_hits<NS, true, false>(c, q, r2max, self);
            } else {
                if (by_id)
                    F.template buffer_hits<NS, false, true>(c, q, r2max, self);
                else
                    F.template buffer_hits<NS, false, false>(c, q, r2max, self);
            }
            if (NL && F.nh > rs) F.add_row(Q, rb_v, t, rs);
        }
    }
}

template <int DIM, int EXCL, bool NL, bool HIST, int ROWS>
__device__ __forceinline__ void fill_chunked(const PairIn& in, const GeomView& G,
                                             const StencilLds& S, const float4* off, int C,
                                             int q0, int q1, Filler<DIM, EXCL, NL, HIST, ROWS>& F)
{
    const int lane = F.lane;
    const float r2max = G.r2max;
    for (int c0 = q0; c0 < q1; c0 += kWave) {
        QueryChunk Q;
        Q.load(in, c0, q1 - c0, lane);
        long long rb_v = 0;
        if (NL && lane < Q.n) rb_v = F.O.offsets[Q.my_id()];
        int w_v = 0;  // entries written so far, per query
        for (int k0 = 0; k0 < C; k0 += kChunkSlots * kWave) {
            Slots<DIM, kChunkSlots> c;
            c.load(in, G.nsten, S, off, k0, C, lane);
            for (int t = 0; t < Q.n; ++t) {
                // Without a list this loop's time depends on where the lines of the instruction
                // cache fall in it, and so on code that has nothing to do with it: dilute
                // droplets, 50,000 points, 1585 us from 16 bytes past a line, 1617 from
                // 48, 1664 to 1681 from 0, 28 and 32.
                if constexpr (!NL) asm volatile(".p2align 6\ns_nop 0\ns_nop 0\ns_nop 0\ns_nop 0");
                const Query q = Q.get<DIM>(t, r2max);
                const long long rbase = NL ? lane_of64(rb_v, t) : 0;
                int w = lane_of(w_v, t);
                if (G.dot)
                    F.template direct_hits<kChunkSlots, true>(c, q, r2max, rbase, w);
                else
                    F.template direct_hits<kChunkSlots, false>(c, q, r2max, rbase, w);
                w_v = lane == t ? w : w_v;
            }
        }
    }
}

inline PairIn make_in(const PairArgs& a)
{
    PairIn in;
    in.cand = a.cand;
    in.cand_start = a.cand_start;
    in.qs = a.qsorted;
    in.q_start = a.q_start;
    return in;
}

inline FillOut make_out(const PairArgs& a, bool hist)
{
    FillOut o;
    o.offsets = a.offsets;
    o.point_idx = a.point_idx;
    o.dist = a.dist;
    o.capacity = a.capacity;
    o.status = a.status;
    o.hist = a.hist;
    o.bins = hist ? a.bins : 0;
    o.r_min = a.r_min;
    o.inv_dr = a.inv_dr;
    return o;
}

}  // namespace

}  // namespace ppa
