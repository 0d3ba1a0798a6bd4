// kernels_graph.hip -- the connectivity the growth produced, as a compact adjacency list,
// and its level-synchronous breadth-first traversal (Sec. 3.4, Figs. 4-5).
//
// A cone that stopped on a target is a connection from the neuron owning the cone to the
// neuron owning the target.  The adjacency list is the paper's pair of arrays: V_a (for
// every neuron the start of its list) and E_a (the lists, neuron after neuron).  Within a
// neuron's list the edges are in increasing cone index, so the list is unique.  It is
// built with the project's stable counting sort of (owner, cone) pairs (kernels_sort.hip;
// non-edges carry the key n_neurons and sort last), a count per neuron and an exclusive
// scan.
//
// The traversal is level-synchronous: a vertex at level d labels its unlabelled neighbours
// d + 1, and the level itself is the frontier flag (a vertex labelled d + 1 is not expanded
// with level d).  A graph whose levels fit a workgroup's LDS is traversed in one launch by one
// workgroup (k_bfs); a larger one takes a launch per level with one thread per vertex, as in
// the paper's kernel.
#include "internal.hpp"

namespace cuesim {

namespace {

constexpr int kGraphThreads = 256;
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kGraphThreads) void k_edge_keys(const int32_t* __restrict__ status,
                                                             const int32_t* __restrict__ owner,
                                                             int n, int n_neurons,
                                                             int32_t* __restrict__ key,
                                                             int32_t* __restrict__ cone,
                                                             int32_t* __restrict__ degree) {
    const int i = blockIdx.x * kGraphThreads + threadIdx.x;
    if (i >= n) return;
    const bool edge = status[i] == kContact;
    key[i] = edge ? owner[i] : n_neurons;
    cone[i] = i;
    if (edge) atomicAdd(&degree[owner[i]], 1);
}

// Exclusive scan of n counts into row_start[0..n] by one workgroup: each thread sums a
// contiguous chunk, the chunk sums are scanned in LDS, then each thread writes its chunk.
__global__ __launch_bounds__(kScanThreads) void k_row_start(const int32_t* __restrict__ degree,
                                                            int n,
                                                            int32_t* __restrict__ row_start) {
    __shared__ int32_t part[kScanThreads];
    const int per = (n + kScanThreads - 1) / kScanThreads;
    const int lo = min((int)threadIdx.x * per, n), hi = min(lo + per, n);
    int32_t sum = 0;
    for (int v = lo; v < hi; ++v) sum += degree[v];
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        const int32_t add = (int)threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    int32_t at = part[threadIdx.x] - sum;
    for (int v = lo; v < hi; ++v) {
        row_start[v] = at;
        at += degree[v];
    }
    if (threadIdx.x == kScanThreads - 1) row_start[n] = part[kScanThreads - 1];
}

__global__ __launch_bounds__(kGraphThreads) void k_fill_edges(
    const int32_t* __restrict__ sorted_cone, const int32_t* __restrict__ target,
    const int32_t* __restrict__ target_owner, const int32_t* __restrict__ row_start,
    int n_neurons, int32_t* __restrict__ edges) {
    const int k = blockIdx.x * kGraphThreads + threadIdx.x;
    if (k >= row_start[n_neurons]) return;
    edges[k] = target_owner[target[sorted_cone[k]]];
}

__global__ __launch_bounds__(kGraphThreads) void k_bfs_level(const int32_t* __restrict__ row_start,
                                                             const int32_t* __restrict__ edges,
                                                             int n, int depth,
                                                             int32_t* __restrict__ level,
                                                             int32_t* __restrict__ grew) {
    const int v = blockIdx.x * kGraphThreads + threadIdx.x;
    if (v >= n || level[v] != depth) return;
    for (int e = row_start[v]; e < row_start[v + 1]; ++e) {
        const int u = edges[e];
        if (level[u] < 0) {
            level[u] = depth + 1;   // every writer writes the same value
            grew[0] = 1;
        }
    }
}

// One launch where the levels fit the LDS (and a vertex 16 bits) and a pass over the edges by
// one workgroup (0.1 us per 1024 edges read again) takes no longer than a launch per level.
constexpr int kBfsMaxVertices = 32768;
constexpr int64_t kBfsMaxEdges = 1 << 18;

// Every level in one launch: the levels in LDS, a thread per edge, a barrier between levels.  A
// level is a pass over the edges, whatever the degrees are: each thread keeps its first
// kBfsHeld edges in registers, both vertices in a word, and reads the others from L2 again,
// kBfsAhead at a time with their loads issued first.  7 levels of 4096 neurons and 25,000 edges:
// 30 us (33 with every edge read again; 196 with a launch per level, its cleared flag and the
// flag read back).
constexpr int kBfsThreads = 1024, kBfsHeld = 32, kBfsAhead = 8;

__global__ __launch_bounds__(kBfsThreads) void k_bfs(const int32_t* __restrict__ from,
                                                     const int32_t* __restrict__ to, int n_edges,
                                                     int n, int root,
                                                     int32_t* __restrict__ level) {
    extern __shared__ int32_t lvl[];
    __shared__ int32_t grew[2];
    const int tid = threadIdx.x;
    // past the end: the last edge again
    auto edge = [&](int e) { return min(e, n_edges - 1); };
    uint32_t held[kBfsHeld];
#pragma unroll
    for (int u = 0; u < kBfsHeld; ++u)
        if (u * kBfsThreads < n_edges) {
            const int e = edge(u * kBfsThreads + tid);
            held[u] = (uint32_t)from[e] << 16 | (uint32_t)to[e];   // n <= kBfsMaxVertices
        }
    for (int v = tid; v < n; v += kBfsThreads) lvl[v] = v == root ? 0 : -1;
    if (tid < 2) grew[tid] = 0;
    __syncthreads();
    for (int depth = 0; depth < n; ++depth) {
        bool any = false;
        auto expand = [&](uint32_t a, uint32_t b) {
            if (lvl[a] == depth && lvl[b] < 0) {
                lvl[b] = depth + 1;   // every writer writes the same value
                any = true;
            }
        };
#pragma unroll
        for (int u = 0; u < kBfsHeld; ++u)
            if (u * kBfsThreads < n_edges) expand(held[u] >> 16, held[u] & 0xffffu);
        for (int e0 = kBfsHeld * kBfsThreads + tid; e0 < n_edges;
             e0 += kBfsThreads * kBfsAhead) {
            int32_t a[kBfsAhead], b[kBfsAhead];
#pragma unroll
            for (int u = 0; u < kBfsAhead; ++u) {
                const int e = edge(e0 + u * kBfsThreads);
                a[u] = from[e];
                b[u] = to[e];
            }
#pragma unroll
            for (int u = 0; u < kBfsAhead; ++u) expand(a[u], b[u]);
        }
        if (any) grew[depth & 1] = 1;
        __syncthreads();
        const bool more = grew[depth & 1] != 0;   // uniform: written before the barrier only
        if (tid == 0) grew[(depth + 1) & 1] = 0;  // last read before that barrier
        __syncthreads();
        if (!more) break;
    }
    for (int v = tid; v < n; v += kBfsThreads) level[v] = lvl[v];
}

__global__ void k_set_root(int32_t* level, int root) {
    if (threadIdx.x == 0) level[root] = 0;
}

int graph_blocks(int n) { return (n + kGraphThreads - 1) / kGraphThreads; }

int key_bits(int n_neurons) {
    int bits = 1;
    while (bits < 31 && (1 << bits) <= n_neurons) ++bits;
    return bits;
}

}  // namespace

hipError_t launch_adjacency(const GraphBuffers& g, const int32_t* status, const int32_t* target,
                            int n_cones, int n_neurons, hipStream_t stream) {
    hipError_t e = hipMemsetAsync(g.degree, 0, (size_t)n_neurons * sizeof(int32_t), stream);
    if (e != hipSuccess) return e;
    const int32_t* sorted_cone = g.cone;
    if (n_cones > 0) {
        hipLaunchKernelGGL(k_edge_keys, dim3(graph_blocks(n_cones)), dim3(kGraphThreads), 0,
                           stream, status, g.owner, n_cones, n_neurons, g.key, g.cone, g.degree);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        bool in_alt = false;
        e = sort_pairs((uint32_t*)g.key, g.cone, (uint32_t*)g.key_sorted, g.cone_sorted,
                       n_cones, key_bits(n_neurons), g.scratch, stream, &in_alt);
        if (e != hipSuccess) return e;
        if (in_alt) sorted_cone = g.cone_sorted;
    }
    hipLaunchKernelGGL(k_row_start, dim3(1), dim3(kScanThreads), 0, stream, g.degree, n_neurons,
                       g.row_start);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (n_cones > 0) {
        hipLaunchKernelGGL(k_fill_edges, dim3(graph_blocks(n_cones)), dim3(kGraphThreads), 0,
                           stream, sorted_cone, target, g.target_owner, g.row_start,
                           n_neurons, g.edges);
        e = hipGetLastError();
    }
    return e;
}

const int32_t* adjacency_from(const GraphBuffers& g) {
    return sort_in_alt(key_bits(g.n_neurons)) ? g.key_sorted : g.key;
}

bool bfs_in_one_launch(int n, int64_t n_edges) {
    return n <= kBfsMaxVertices && n_edges <= kBfsMaxEdges;
}

hipError_t launch_bfs(const GraphBuffers& g, int n_edges, int root, hipStream_t stream) {
    const size_t lds = (size_t)g.n_neurons * sizeof(int32_t);
    hipError_t e = hipFuncSetAttribute((const void*)k_bfs,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kBfsMaxVertices * (int)sizeof(int32_t));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bfs, dim3(1), dim3(kBfsThreads), lds, stream, adjacency_from(g), g.edges,
                       n_edges, g.n_neurons, root, g.level);
    return hipGetLastError();
}

hipError_t launch_bfs_init(int32_t* level, int n, int root, hipStream_t stream) {
    hipError_t e = hipMemsetAsync(level, 0xFF, (size_t)n * sizeof(int32_t), stream);   // -1
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_set_root, dim3(1), dim3(64), 0, stream, level, root);
    return hipGetLastError();
}

hipError_t launch_bfs_level(const int32_t* row_start, const int32_t* edges, int n, int depth,
                            int32_t* level, int32_t* grew, hipStream_t stream) {
    hipLaunchKernelGGL(k_bfs_level, dim3(graph_blocks(n)), dim3(kGraphThreads), 0, stream,
                       row_start, edges, n, depth, level, grew);
    return hipGetLastError();
}

}  // namespace cuesim
