// Work distribution of the batched pair passes: per-XCD queues of home cells
// and the geometry of a frame.
#pragma once

#include "pair_list.hpp"

namespace ppa {

namespace {

// ---------------------------------------------------------------------------
// Batch: the same passes over the cells of many frames at once.  The home
// cells of all frames form one global range, cut into runs of B.run
// consecutive cells; a wavefront switches geometry (grid, stencil offsets,
// frame-local point indices, the frame's histogram) when a run takes it into
// another frame.
// ---------------------------------------------------------------------------
// Work queues of a batch pass.  The work items (cells, or parts of them) of
// XCD x (workgroups are dispatched round-robin over the 8 XCDs) are
// [x I / 8, (x + 1) I / 8); they are handed out in order, in runs, by an
// atomic counter, so the runs in flight on an XCD are neighbours sharing
// stencil cells in its L2, and a wavefront that finds its own XCD's queue
// empty takes runs from the other XCDs' queues, so uneven frames (cheap and
// dear cells) finish together.  Every wavefront ends when all eight queues
// are empty.
//
// Runs are B.run items long (fewer when there are not PER such runs per
// wavefront) until two runs per wavefront of the XCD are left, then halve
// once per wavefront, down to single items: a run of 16
// full cells takes a wavefront about 0.4 ms, so without the taper the last
// runs leave most of the chip idle.  Draws are atomics on memory shared by
// the XCDs, about 12 ns each on one line: each counter has its own 128-byte
// line, a wavefront's first run is the one of its own number, the next run is
// drawn before the current one is worked, and a wavefront whose queue is empty
// reads all counters at once instead of drawing from each (that alone cost
// eight serialised draws per wavefront).
// 96 frames, 1.2 M points, 62 M pairs: count 643 -> 214 us, fill 1233 -> 566
// us (two first runs per wavefront instead of eight: 225 and 762 us); with the
// first run not drawn and the first frame probes kept, count 196 -> 186 us.
// PER is 8 in the count pass, whose cells are short against a draw (at 16 the
// frames above go cell by cell: 265 us), and 32 in the fill pass, whose last
// runs cost more than its draws: a batch of 256 frames, 11 M points, at most 16
// cells a run, 6.08 -> 5.76 ms with 32 instead of 8.
template <int PER>
struct RunQueue {
    int x;       // XCD whose queue is being drained
    int c0, n;   // that XCD's first item, and its items
    int waves;   // wavefronts per XCD
    unsigned long long pend;  // lane 0: the draw made ahead

    // Items of the k-th run of a queue of n items: [t, t + len); t >= n past the end.
    static __device__ __forceinline__ int run_at(int run, int waves, int n, long long k, int& len)
    {
        run = max(1, min(run, n / (PER * waves)));
        const long long whole = max(0LL, ((long long)n - 2LL * waves * run) / run);
        len = run;
        if (k < whole) return (int)(k * run);
        k -= whole;
        long long t = whole * run;
        while (k >= waves && len > 1) {
            t += (long long)waves * len;
            k -= waves;
            len >>= 1;
        }
        t += k * len;
        return (int)(t < n ? t : n);
    }
    // The first item of XCD x's queue.
    static __device__ __forceinline__ int first(const BatchGeom& B, int x)
    {
        return (int)((long long)x * B.ncells * B.split / 8);
    }
    __device__ __forceinline__ void set(const BatchGeom& B, int xcd)
    {
        x = xcd;
        c0 = first(B, x);
        n = first(B, x + 1) - c0;
    }
    __device__ __forceinline__ void draw(unsigned long long* queue, int lane)
    {
        if (lane == 0) pend = waves + atomicAdd(&queue[x * kQueueStride], 1ull);
    }
    // A wavefront's first run is the one of its own number within the XCD.
    __device__ __forceinline__ void start(const BatchGeom& B, int wpb, int wv)
    {
        waves = (int)(gridDim.x >> 3) * wpb;
        pend = (unsigned long long)((blockIdx.x >> 3) * wpb + wv);
        set(B, blockIdx.x & 7);
    }
    // The next run [t, te) for this wavefront; false when every queue is empty.
    __device__ __forceinline__ bool next(const BatchGeom& B, unsigned long long* queue, int lane,
                                         int& t, int& te)
    {
        for (;;) {
            const long long k = (long long)uniform64(pend);
            int len;
            const int at = run_at(B.run, waves, n, k, len);
            if (at < n) {
                draw(queue, lane);
                t = c0 + at;
                te = t + min(len, n - at);
                return true;
            }
            // this queue is empty: the next one that is not, in cyclic order
            bool open = false;
            if (lane < 8) {
                const int y = (x + 1 + lane) & 7;
                const int m = first(B, y + 1) - first(B, y);
                const unsigned long long d = __hip_atomic_load(
                    &queue[y * kQueueStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                open = run_at(B.run, waves, m, waves + (long long)d, len) < m;
            }
            const unsigned long long some = __ballot(open);
            if (!some) return false;
            set(B, (x + __ffsll((long long)some)) & 7);
            draw(queue, lane);
        }
    }
};

// Frame of a global cell: the last f with cell_base[f] <= tile, by a 64-way
// search (the lanes probe 64 evenly spaced frames at once; a binary search
// would chain a dependent read of memory per halving).  The first probes are
// the same for every cell and stay in a register.
struct FrameSearch {
    int step, base;

    __device__ __forceinline__ FrameSearch(const BatchGeom& B, int lane)
    {
        step = (B.nframes + kWave - 1) / kWave;
        base = lane * step < B.nframes ? B.cell_base[lane * step] : INT_MAX;
    }
    __device__ __forceinline__ int find(const BatchGeom& B, int tile, int lane) const
    {
        // lane 0 always probes a frame at or below
        int lo = (__popcll(__ballot(base <= tile)) - 1) * step;
        int n = min(step, B.nframes - lo);  // the frame lies in [lo, lo + n)
        while (n > 1) {
            const int st = (n + kWave - 1) / kWave;
            const bool at = lane * st < n && B.cell_base[lo + lane * st] <= tile;
            const int hit = __popcll(__ballot(at)) - 1;
            lo += hit * st;
            n = min(st, n - hit * st);
        }
        return uniform(lo);
    }
};

// Loads frame f's geometry: the view in scalar registers, the stencil
// offsets into this wavefront's LDS.
__device__ __forceinline__ GeomView load_frame(const BatchGeom& B, int f, float4* off, int lane)
{
    const FrameInfo& F = B.frames[f];
    GeomView v;
    v.n0 = uniform(F.box.ni[0]);
    v.n1 = uniform(F.box.ni[1]);
    v.n2 = uniform(F.box.ni[2]);
    v.nsten = uniform(F.nsten);
    v.cell_base = uniform(F.cell_base);
    v.r2max = B.r2max;
    v.dot = uniform(F.dot);
    if (lane < 27) off[lane] = make_float4(F.off[lane][0], F.off[lane][1], F.off[lane][2], 0.f);
    wave_sync();
    return v;
}

// Workgroups for a batch pass: as many as fit at once (times the cap per CU
// when one is set), a multiple of 8; the queues hand out the work.
template <typename K>
inline int batch_blocks(K kernel, int threads, size_t lds, int blocks_cap)
{
    const int cus = device_cus();
    int per_cu = resident_per_cu(kernel, threads, lds);
    if (blocks_cap > 0 && per_cu > blocks_cap) per_cu = blocks_cap;
    return (cus * per_cu + 7) / 8 * 8;
}

}  // namespace

}  // namespace ppa
