// Clusters of the cluster module (the paper's analysis modules: cluster
// membership is defined by neighbour bonds): the connected components of
// the undirected graph on n points whose edges are the pairs of a
// NeighborList.  labels[i] is the smallest point index of i's component;
// optional outputs number the components in order of that index
// (cluster_idx), count their points (sizes) and count them (n_clusters).
//
// Union-find over the labels array as the parent forest.  A seed pass
// points every point at its smallest listed neighbour; hooking rounds over
// the bonds (the root of a point's component pointed at the smallest label
// among the point's neighbours, by plain stores of which any may win)
// alternate with passes that point every node at its root, until a round
// changes nothing, so the
// large components form flat; a last lock-free union pass over every bond makes
// the result exact, most bonds ending with two equal labels.  Finds in the union
// passes halve paths with plain stores; the compress passes only read the forest
// and write their own entries.  A union finds
// both roots and links the larger under the smaller with a compare-and-swap
// on the larger root's parent; a failed swap means that root was linked
// meanwhile, and the union continues from its new parent.  Parents only
// ever point to smaller indices, so the root of a component is its smallest
// index, every find ends, and the larger of the two roots a union works on
// shrinks on every retry, so every union ends.  A compress pass sets every
// label to its root, each lane writing only its own entry (by atomic
// minimum, which keeps a root a concurrent union may have written); the
// compact numbering is a scan over the roots.  What bounds it: reads of
// labels at random places and, where a pass needs them, atomics (to one
// address about 12 ns each, serialised across the XCDs; to scattered ones
// about 5 per ns).  For a list the caller declares
// symmetric, later rounds sample two bonds per row and the union pass skips the
// points of the largest sampled component (their bonds to other points are
// in those points' rows).
#include "internal.hpp"

namespace ppa {

namespace {

constexpr int kClBlock = 256;
constexpr int kClRounds = kClusterRounds;  // hooking rounds at most
constexpr int kClFirst = 4;                // bonds per row of the first round (symmetric lists)
constexpr int kClSampled = 2;              // and of the later ones

__device__ __forceinline__ int parent_of(int* p, int x)
{
    return __hip_atomic_load(&p[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A label read through the caches, and a parent written through them (the
// hooking rounds: racing lanes, no ordering needed; a word is never torn).
__device__ __forceinline__ int parent_cached(int* p, int x)
{
    return __hip_atomic_load(&p[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void set_parent(int* p, int x, int v)
{
    __hip_atomic_store(&p[x], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Root of x, without writes: the lanes of a large component all walk
// through the few nodes near its root, and writes there would serialise.
__device__ __forceinline__ int root_of(int* p, int x)
{
    int px;
    while ((px = parent_of(p, x)) != x) x = px;
    return x;
}

// Root of x, halving the path on the way (the union passes): each visited
// node is pointed at its grandparent by a plain store.  Only non-roots are
// written, every value is an ancestor, and no other kind of write to a
// non-root happens during a union pass, so the forest stays valid.
__device__ __forceinline__ int root_halving(int* p, int x)
{
    while (true) {
        const int px = parent_of(p, x);
        if (px == x) return x;
        const int gp = parent_of(p, px);
        if (gp == px) return px;
        __hip_atomic_store(&p[x], gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = gp;
    }
}

// Joins the trees of a and b; returns their common root.
__device__ int unite(int* p, int a, int b)
{
    while (true) {
        a = root_halving(p, a);
        b = root_halving(p, b);
        if (a == b) return a;
        if (a < b) {
            const int t = a;
            a = b;
            b = t;
        }
        // a > b: hang root a under b unless a stopped being a root
        const int old = atomicCAS(&p[a], a, b);
        if (old == a) return b;
        a = old;
    }
}

// Zeroes `words` 32-bit words at z (status, scan state) and words2 at z2 (sizes).
__global__ void __launch_bounds__(kClBlock) cl_init_kernel(unsigned* z, long long words,
                                                           unsigned* z2, long long words2)
{
    const long long stride = (long long)gridDim.x * kClBlock;
    const long long t = (long long)blockIdx.x * kClBlock + threadIdx.x;
    for (long long i = t; i < words; i += stride) z[i] = 0u;
    for (long long i = t; i < words2; i += stride) z2[i] = 0u;
}

// Checked bounds of row i of the list (empty when the row is invalid).
__device__ __forceinline__ bool row_bounds(const int64_t* offsets, int i, long long capacity,
                                           unsigned* status, long long& e0, long long& e1)
{
    e0 = offsets[i];
    e1 = offsets[i + 1];
    if (e0 < 0 || e1 < e0 || e1 > capacity) {
        atomicOr(status, kStatusBadList);
        e0 = e1 = 0;
        return false;
    }
    return true;
}

// Four consecutive neighbours of a row from bond e (the last one repeated
// past the row's end), read together so that their latencies overlap.
__device__ __forceinline__ void four_bonds(const int32_t* __restrict__ idx, long long e,
                                           long long e1, int (&j)[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) j[k] = idx[e + k < e1 ? e + k : e1 - 1];
}

// First links: every point to the smallest of itself and its listed
// neighbours (each lane writes only its own parent, a smaller index, so the
// result is a valid forest of unions without any atomics).
__global__ void __launch_bounds__(kClBlock) cl_seed_kernel(const int64_t* __restrict__ offsets,
                                                           const int32_t* __restrict__ idx, int n,
                                                           long long capacity, int* labels,
                                                           unsigned* status)
{
    const int i = blockIdx.x * kClBlock + threadIdx.x;
    if (i >= n) return;
    long long e0, e1;
    row_bounds(offsets, i, capacity, status, e0, e1);
    int m = i;
    for (long long e = e0; e < e1; e += 4) {
        int j[4];
        four_bonds(idx, e, e1, j);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (j[k] < 0 || j[k] >= n) {
                atomicOr(status, kStatusBadList);
                continue;
            }
            m = j[k] < m ? j[k] : m;
        }
    }
    labels[i] = m;
}

// One hooking round over every bond (first > 0: the first `first` bonds of a
// row): the root of point i is pointed at the smallest label among i's
// neighbours; with BOTH (a list that may hold a bond in one row only) the
// root of a neighbour with a larger label is also pointed at i's.  Labels
// are flat here (every label is a root).  A hook is a plain store: of
// several hooks of one root any may win, and each joins bonded points and
// keeps the parent below its node, so the forest stays a valid subset of the
// components, and every root that has a smaller neighbour is hooked; later
// rounds and the closing union pass join what was left.  Atomic minima
// instead cost 165 us a round (2^20 points, about 5 per ns across the XCDs),
// and only choose which smaller neighbour a root hangs under.
template <bool BOTH>
__global__ void __launch_bounds__(kClBlock) cl_sv_kernel(const int64_t* __restrict__ offsets,
                                                         const int32_t* __restrict__ idx, int n,
                                                         long long capacity, int first,
                                                         int* labels, const int* prev_changed,
                                                         int* changed)
{
    // nothing moved in the previous round: the forest has converged
    if (prev_changed && __hip_atomic_load(prev_changed, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) == 0)
        return;
    const int i = blockIdx.x * kClBlock + threadIdx.x;
    if (i >= n) return;
    long long e0 = offsets[i], e1 = offsets[i + 1];
    if (e0 < 0 || e1 < e0 || e1 > capacity) return;
    if (first > 0 && e1 > e0 + first) e1 = e0 + first;  // a sample of the bonds
    // cached loads: a stale label is an older ancestor, which only makes a
    // hook weaker; the closing union pass is exact either way
    const int li = parent_cached(labels, i);
    int m = li;
    bool moved = false;
    for (long long e = e0; e < e1; e += 4) {
        int j[4], l[4];
        four_bonds(idx, e, e1, j);
#pragma unroll
        for (int k = 0; k < 4; ++k) l[k] = j[k] < 0 || j[k] >= n ? li : parent_cached(labels, j[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            m = l[k] < m ? l[k] : m;
            if (BOTH && l[k] > li && parent_cached(labels, l[k]) > li) {
                set_parent(labels, l[k], li);
                moved = true;
            }
        }
    }
    // read first: in a large component the target is one shared root
    if (m < li && parent_cached(labels, li) > m) {
        set_parent(labels, li, m);
        moved = true;
    }
    const unsigned long long any = __ballot(moved);
    if (any && (threadIdx.x & (warpSize - 1)) == __ffsll((long long)any) - 1)
        __hip_atomic_store(changed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Unites point i with its neighbours.
__global__ void __launch_bounds__(kClBlock) cl_hook_kernel(const int64_t* __restrict__ offsets,
                                                           const int32_t* __restrict__ idx, int n,
                                                           long long capacity,
                                                           const int* giant, int* labels)
{
    const int i = blockIdx.x * kClBlock + threadIdx.x;
    if (i >= n) return;
    // a symmetric list: a point already in the sampled largest component
    // leaves its bonds to the other ends (a bond to a point outside is in
    // that point's row; a bond inside joins nothing new)
    int li = parent_cached(labels, i);
    if (giant && li == *giant) return;
    // bounds were checked (and reported) by the seed pass
    long long e0 = offsets[i], e1 = offsets[i + 1];
    if (e0 < 0 || e1 < e0 || e1 > capacity) return;
    // Two points with one label are joined already, however stale the labels are:
    // a label is a point of the same tree.  Without this test every bond reads
    // its root through the caches, and the roots of the components that the
    // rounds left apart are a few lines that the whole chip waits for (a ladder
    // of 2^20 points in random order 8174 us, 837 now; uniform 2D points past
    // percolation 3659 and 558).
    for (long long e = e0; e < e1; ++e) {
        const int j = idx[e];
        if (j < 0 || j >= n || j == i) continue;
        const int lj = parent_cached(labels, j);
        if (lj != li) li = unite(labels, li, lj);
    }
}

// The root most of kClSamples evenly spaced points share (ties: the smaller
// root), after a compress pass: one workgroup, the samples counted by root
// in an LDS table (kClSamples roots fit; a sample whose probe sequence is
// full is left out, which only makes the choice less representative).
constexpr int kClSamples = 1024;
constexpr int kClTable = 2048;
constexpr int kClProbes = 16;

__global__ void __launch_bounds__(kClSamples) cl_giant_kernel(int n, const int* labels, int* giant)
{
    __shared__ int s_root[kClTable], s_count[kClTable];
    __shared__ unsigned long long s_best[kClSamples / 64];
    const int t = threadIdx.x;
    for (int k = t; k < kClTable; k += kClSamples) {
        s_root[k] = -1;
        s_count[k] = 0;
    }
    __syncthreads();
    const int lab = labels[(int)(((long long)t * n) / kClSamples)];
    unsigned h = (unsigned)lab * 2654435761u >> 21;  // 11 bits: kClTable slots
    static_assert(kClTable == 1 << 11, "the hash above gives 11 bits");
    for (int p = 0; p < kClProbes; ++p) {
        const int old = atomicCAS(&s_root[h], -1, lab);
        if (old == -1 || old == lab) {
            atomicAdd(&s_count[h], 1);
            break;
        }
        h = (h + 1) & (kClTable - 1);
    }
    __syncthreads();
    // largest count first, then smallest root: one 64-bit key per slot
    unsigned long long key = 0;
    for (int k = t; k < kClTable; k += kClSamples)
        if (s_root[k] >= 0) {
            const unsigned long long o = ((unsigned long long)(unsigned)s_count[k] << 32) |
                                         (unsigned)(0x7fffffff - s_root[k]);
            key = o > key ? o : key;
        }
    for (int sh = 32; sh > 0; sh >>= 1) {
        const unsigned long long o = __shfl_xor(key, sh);
        key = o > key ? o : key;
    }
    if ((t & 63) == 0) s_best[t >> 6] = key;
    __syncthreads();
    if (t == 0) {
        unsigned long long b = s_best[0];
        for (int w = 1; w < kClSamples / 64; ++w) b = s_best[w] > b ? s_best[w] : b;
        *giant = 0x7fffffff - (int)(unsigned)(b & 0xffffffffull);
    }
}

__global__ void __launch_bounds__(kClBlock) cl_compress_kernel(int n, int* labels, int* is_root,
                                                               const int* changed)
{
    if (changed && __hip_atomic_load(changed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
        return;  // the hooking round before changed nothing
    const int i = blockIdx.x * kClBlock + threadIdx.x;
    if (i >= n) return;
    // each lane writes only its own entry; the minimum keeps a root that a
    // union may have written since (no other lane writes this entry here).
    // Between hooking rounds a cached walk is enough (a stale root is still
    // an ancestor); the last pass reads coherently.
    int r;
    if (changed) {
        int x = i, px;
        while ((px = labels[x]) != x) x = px;
        r = x;
    } else {
        r = root_of(labels, i);
    }
    atomicMin(&labels[i], r);
    if (is_root) is_root[i] = r == i ? 1 : 0;
}

constexpr int kClIndexBlock = 1024;

__global__ void __launch_bounds__(kClIndexBlock) cl_index_kernel(int n,
                                                                 const int* __restrict__ labels,
                                                                 const int64_t* __restrict__ rank,
                                                                 int32_t* cluster_idx,
                                                                 int32_t* sizes)
{
    __shared__ int s_c[kClIndexBlock / 64], s_n[kClIndexBlock / 64];
    const int i = blockIdx.x * kClIndexBlock + threadIdx.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const bool live = i < n;
    const int c = live ? (int)rank[labels[i]] : -1;
    if (live && cluster_idx) cluster_idx[i] = c;
    if (!sizes) return;
    // the cluster of each wavefront's first point is counted for the whole
    // workgroup: the wavefronts that share it (all of them inside a large
    // cluster) add one total with one atomic
    const int c0 = __builtin_amdgcn_readfirstlane(c);
    const unsigned long long m0 = __ballot(live && c == c0);
    if (lane == 0) {
        s_c[wv] = c0;
        s_n[wv] = __popcll(m0);
    }
    __syncthreads();
    if (threadIdx.x < kClIndexBlock / 64) {
        const int w = threadIdx.x;
        // the first wavefront holding this cluster adds for all that hold it
        int first = w, total = 0;
        for (int u = 0; u < kClIndexBlock / 64; ++u)
            if (s_c[u] == s_c[w]) {
                if (u < first) first = u;
                total += s_n[u];
            }
        if (first == w && s_c[w] >= 0 && total > 0) atomicAdd(&sizes[s_c[w]], total);
    }
    // the other points: one atomic per distinct cluster of the wavefront for
    // three more rounds, then one by one
    bool done = !live || c == c0;
    for (int round = 0; round < 3; ++round) {
        const unsigned long long pend = __ballot(!done);
        if (!pend) break;
        const int cr = __builtin_amdgcn_readlane(c, __ffsll((unsigned long long)pend) - 1);
        const unsigned long long m = __ballot(!done && c == cr);
        if (!done && c == cr) {
            const unsigned below = __builtin_amdgcn_mbcnt_hi(
                (unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            if (below == 0) atomicAdd(&sizes[cr], __popcll(m));
            done = true;
        }
    }
    if (!done) atomicAdd(&sizes[c], 1);
}

inline int blocks_for(long long n) { return (int)((n + kClBlock - 1) / kClBlock); }

}  // namespace

void launch_cluster(const ClusterArgs& a, hipStream_t s)
{
    const int n = (int)a.n;
    const bool ranks = a.cluster_idx || a.sizes || a.n_clusters;
    const long long zwords = (long long)(a.zero_bytes / 4);
    const long long swords = a.sizes ? (long long)n : 0;
    const long long most = zwords > swords ? zwords : swords;
    const int ib = (int)(most < 1 ? 1 : (blocks_for(most) < 4096 ? blocks_for(most) : 4096));
    hipLaunchKernelGGL(cl_init_kernel, dim3(ib), dim3(kClBlock), 0, s, a.zero, zwords,
                       (unsigned*)a.sizes, swords);
    if (n == 0) return;
    const int nb = blocks_for(n);
    hipLaunchKernelGGL(cl_seed_kernel, dim3(nb), dim3(kClBlock), 0, s, a.offsets, a.idx, n,
                       a.capacity, a.labels, a.status);
    hipLaunchKernelGGL(cl_compress_kernel, dim3(nb), dim3(kClBlock), 0, s, n, a.labels, nullptr,
                       nullptr);
    // hooking rounds, each flattened, until one changes nothing (later
    // rounds then return at once: no host synchronisation); then the union
    // pass over every bond makes the result exact whatever the rounds left
    // sparse lists (below about 3 bonds per point, under the percolation
    // threshold of random geometric graphs) form no large component: the
    // union pass alone is faster there
    // With a symmetric list (every bond in both rows) the rounds hook only
    // the first bonds of each row; the root most sampled points share then
    // marks the largest component, whose points the union pass skips (the
    // sampling of the Afforest method).  2^20-point uniform system, r = 1.2
    // (7.2 bonds a point): 1164 us with rounds of one atomic minimum per
    // bond, 305 us now; r = 0.95, at percolation: 1294 and 350 us.
    const int rounds = a.capacity < 3 * (long long)n ? 0 : kClRounds;
    for (int r = 0; r < rounds; ++r) {
        const int* prev = r > 0 ? a.round_flags + (r - 1) : nullptr;
        // the first round sees small components (a seed tree holds about a
        // row's points) and takes four bonds per row; after it a component is
        // large enough that two reach its neighbours (every bond in the first
        // round: 333 us instead of 309 below)
        const int first = a.symmetric ? (r == 0 ? kClFirst : kClSampled) : 0;
        if (a.symmetric)
            hipLaunchKernelGGL(cl_sv_kernel<false>, dim3(nb), dim3(kClBlock), 0, s, a.offsets,
                               a.idx, n, a.capacity, first, a.labels, prev, a.round_flags + r);
        else
            hipLaunchKernelGGL(cl_sv_kernel<true>, dim3(nb), dim3(kClBlock), 0, s, a.offsets,
                               a.idx, n, a.capacity, first, a.labels, prev, a.round_flags + r);
        hipLaunchKernelGGL(cl_compress_kernel, dim3(nb), dim3(kClBlock), 0, s, n, a.labels,
                           nullptr, a.round_flags + r);
    }
    const bool skip_giant = a.symmetric && rounds > 0;  // no large component without rounds
    if (skip_giant) {
        // the last round's compress read a cached walk: one exact pass first
        hipLaunchKernelGGL(cl_compress_kernel, dim3(nb), dim3(kClBlock), 0, s, n, a.labels,
                           nullptr, nullptr);
        hipLaunchKernelGGL(cl_giant_kernel, dim3(1), dim3(kClSamples), 0, s, n, a.labels,
                           a.giant);
    }
    hipLaunchKernelGGL(cl_hook_kernel, dim3(nb), dim3(kClBlock), 0, s, a.offsets, a.idx, n,
                       a.capacity, skip_giant ? a.giant : nullptr, a.labels);
    hipLaunchKernelGGL(cl_compress_kernel, dim3(nb), dim3(kClBlock), 0, s, n, a.labels,
                       ranks ? a.is_root : nullptr, nullptr);
    if (!ranks) return;
    launch_scan_i64_total(a.is_root, a.rank, n, a.scan_flags, a.ticket,
                          (unsigned long long*)a.n_clusters, s);
    if (a.cluster_idx || a.sizes)
        hipLaunchKernelGGL(cl_index_kernel, dim3((n + kClIndexBlock - 1) / kClIndexBlock),
                           dim3(kClIndexBlock), 0, s, n, a.labels,
                           a.rank, a.cluster_idx, a.sizes);
}

}  // namespace ppa
