// Residency-octree maintenance (Sec. 5.2, Sec. 5.3): metadata reduction,
// incremental residency update with early-stopping OR propagation, and
// from-scratch rebuild.
#include <string.h>

#include <algorithm>

#include "common.h"

namespace ro {

// Child index range of a level-d node: children per axis are 1 or 2.
__device__ inline void child_range(const TreeGeo &t, int d, uint32_t x, uint32_t y, uint32_t z, uint32_t c0[3],
                                   uint32_t cn[3]) {
    const uint32_t p[3] = {x, y, z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int r = t.nlog[d + 1][a] - t.nlog[d][a];
        c0[a] = p[a] << r;
        cn[a] = 1u << r;
    }
}

__device__ inline void node_coords(const TreeGeo &t, int d, uint64_t i, uint32_t *x, uint32_t *y, uint32_t *z) {
    *x = (uint32_t)(i & ((1u << t.nlog[d][0]) - 1));
    *y = (uint32_t)((i >> t.nlog[d][0]) & ((1u << t.nlog[d][1]) - 1));
    *z = (uint32_t)(i >> (t.nlog[d][0] + t.nlog[d][1]));
}

// Children of node i of level d in an array of their level, 2^gl entries per
// node, this lane's the `lane`-th; `none` past the last child.  An axis of one
// child takes no bit of k.
template <typename T>
__device__ inline void lds_children(const TreeGeo &t, int d, uint32_t i, int gl, uint32_t lane, const T *lv,
                                    uint32_t none, uint32_t v[8]) {
    uint32_t x, y, z, c0[3], cn[3];
    node_coords(t, d, i, &x, &y, &z);
    child_range(t, d, x, y, z, c0, cn);
    const uint32_t n = cn[0] * cn[1] * cn[2], lx = cn[0] >> 1, ly = lx + (cn[1] >> 1);
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)
        v[k] = k < n ? (uint32_t)lv[((node_index(t, d + 1, c0[0] + (k & (cn[0] - 1)),
                                                 c0[1] + ((k >> lx) & (cn[1] - 1)), c0[2] + (k >> ly)) -
                                      t.noff[d + 1])
                                     << gl) +
                                    lane]
                     : none;
}

static __host__ __device__ inline uint64_t level_nodes(const TreeGeo &t, int d) {
    return 1ull << (t.nlog[d][0] + t.nlog[d][1] + t.nlog[d][2]);
}

static inline unsigned nblocks(uint64_t n) { return (unsigned)((n + 255) / 256); }

// Nodes of the deepest level that one block takes through to the root in one
// launch, the levels above it from LDS (a round trip to memory per level took
// 14 us for the residency masks, as long as the launches it replaced).  A
// level of 512 nodes is two turns of 1024 lanes at 16 channels.
constexpr uint32_t kTopNodes = 512;

// Lanes per node (log2): one per channel, so that a node's row is read and
// written as one piece and its lanes are in one wave.
static inline int lanes_log(int m) {
    int gl = 0;
    while ((1 << gl) < m) ++gl;
    return gl;
}
static_assert(kMaxC <= 64, "a node's channels are lanes of one wave");

// Deepest level below the leaves' parents that the one-block kernels start
// from (-1: none).
static inline int top_level(const TreeGeo &t, int from) {
    int d = from;
    while (d >= 0 && level_nodes(t, d) > kTopNodes) --d;
    return d;
}

// [min, max] of leaf li from the caller's array, as a metadata word; `wide`:
// the array is 4-byte aligned.
__device__ inline uint32_t leaf_word(const uint16_t *__restrict__ leaf_mm, bool wide, uint64_t li) {
    if (wide) return ((const uint32_t *)leaf_mm)[li];
    return (uint32_t)leaf_mm[2 * li] | (uint32_t)leaf_mm[2 * li + 1] << 16;
}

// Leaf metadata of channel c: from the caller's [n_leaves][2] array (level
// 0), or, with leaf_mm null, unknown ([0, unknown_max], level unknown).  One
// word of every node's row of m: a partial write of a memory line costs the
// line read and written (8.4 million rows of 64 bytes: 221 us, as for whole
// rows), a read alone 85 us, so a word that is there already is not written
// again (the background is empty in every channel).
__global__ __launch_bounds__(256) void k_meta_leaf(const uint16_t *__restrict__ leaf_mm, bool wide,
                                                   uint32_t *__restrict__ meta, uint8_t *__restrict__ level,
                                                   uint64_t n_leaves, uint32_t leaf_off, int m, int c,
                                                   uint32_t unknown_max) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_leaves) return;
    const uint32_t v = leaf_mm ? leaf_word(leaf_mm, wide, i) : unknown_max << 16;
    const uint8_t lev = leaf_mm ? 0 : (uint8_t)kLevelUnknown;
    uint32_t *p = meta + ((uint64_t)leaf_off + i) * m + c;
    uint8_t *q = level + i * m + c;
    if (*p != v) *p = v;
    if (*q != lev) *q = lev;
}

// The leaves' parents of channel c, from the caller's array (4 bytes a leaf)
// and not from the rows just written (a line a leaf: 188 us for the same
// 8.4 million).
__global__ __launch_bounds__(256) void k_meta_parent(TreeGeo t, const uint16_t *__restrict__ leaf_mm, bool wide,
                                                     uint32_t *__restrict__ meta, int m, int c,
                                                     uint32_t unknown_max) {
    const int D = t.depth, d = D - 1;
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= level_nodes(t, d)) return;
    uint32_t x, y, z, c0[3], cn[3];
    node_coords(t, d, i, &x, &y, &z);
    child_range(t, d, x, y, z, c0, cn);
    uint32_t mn = leaf_mm ? 0xFFFFu : 0u, mx = leaf_mm ? 0u : unknown_max;
    if (leaf_mm) {
        const uint32_t n = cn[0] * cn[1] * cn[2], lx = cn[0] >> 1, ly = lx + (cn[1] >> 1);
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {  // an axis of one child takes no bit of k
            const uint32_t kk = k < n ? k : 0;
            const uint32_t v = leaf_word(leaf_mm, wide,
                                         node_index(t, D, c0[0] + (kk & (cn[0] - 1)),
                                                    c0[1] + ((kk >> lx) & (cn[1] - 1)), c0[2] + (kk >> ly)) -
                                             t.noff[D]);
            mn = min(mn, v & 0xFFFFu);
            mx = max(mx, v >> 16);
        }
    }
    uint32_t *p = meta + ((uint64_t)t.noff[d] + i) * m + c;
    const uint32_t v = mn | (mx << 16);
    if (*p != v) *p = v;
}

// Children of node i of level d in channel c, and their reduction: min of the
// mins, max of the maxes.
__device__ inline void meta_load(const TreeGeo &t, int d, uint64_t i, const uint32_t *meta, int m, int c,
                                 uint32_t v[8]) {
    uint32_t x, y, z, c0[3], cn[3];
    node_coords(t, d, i, &x, &y, &z);
    child_range(t, d, x, y, z, c0, cn);
    const uint32_t n = cn[0] * cn[1] * cn[2], lx = cn[0] >> 1, ly = lx + (cn[1] >> 1);
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)  // an axis of one child takes no bit of k
        v[k] = k < n ? meta[(uint64_t)node_index(t, d + 1, c0[0] + (k & (cn[0] - 1)),
                                                 c0[1] + ((k >> lx) & (cn[1] - 1)), c0[2] + (k >> ly)) * m + c]
                     : 0x0000FFFFu;
}

__device__ inline uint32_t meta_of(const uint32_t v[8]) {
    uint32_t mn = 0xFFFFu, mx = 0;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
        mn = min(mn, v[k] & 0xFFFFu);
        mx = max(mx, v[k] >> 16);
    }
    return mn | (mx << 16);
}

// Parents of level d: 2^gl lanes per node over the channels from c_first of
// `chans` (bit c = channel c).
__global__ __launch_bounds__(256) void k_meta_reduce(TreeGeo t, int d, uint32_t *__restrict__ meta, int m, int gl,
                                                     int c_first, uint32_t chans) {
    const uint64_t tid = (uint64_t)blockIdx.x * 256 + threadIdx.x, i = tid >> gl;
    const int c = c_first + (int)(tid & ((1u << gl) - 1));
    if (i >= level_nodes(t, d) || c >= m || !(chans >> c & 1u)) return;
    uint32_t v[8];
    meta_load(t, d, i, meta, m, c, v);
    meta[((uint64_t)t.noff[d] + i) * m + c] = meta_of(v);
}

// Levels d, d - 1, .. 0 by one block: the deepest one from memory, four nodes
// of a lane at a time with all their loads issued first, the others from LDS.
__global__ __launch_bounds__(1024) void k_meta_top(TreeGeo t, int d, uint32_t *meta, int m, int gl, int c_first,
                                                   uint32_t chans) {
    __shared__ uint32_t lv[2][kTopNodes * kMaxC];
    const uint32_t lane = threadIdx.x & ((1u << gl) - 1), step = 1024u >> gl;  // nodes a round
    const int c = c_first + (int)lane;
    const bool on = c < m && (chans >> c & 1u);
    const uint32_t n0 = (uint32_t)level_nodes(t, d);
    for (uint32_t i0 = threadIdx.x >> gl; i0 < n0; i0 += 4 * step) {
        uint32_t v[4][8];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r)
            if (on && i0 + r * step < n0) meta_load(t, d, i0 + r * step, meta, m, c, v[r]);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = i0 + r * step;
            if (!on || i >= n0) continue;
            const uint32_t w = meta_of(v[r]);
            meta[((uint64_t)t.noff[d] + i) * m + c] = w;
            lv[0][(i << gl) + lane] = w;
        }
    }
    int from = 0;
    for (--d; d >= 0; --d, from ^= 1) {
        __syncthreads();
        const uint32_t n = (uint32_t)level_nodes(t, d);
        for (uint32_t i = threadIdx.x >> gl; i < n; i += step) {
            if (!on) continue;
            uint32_t v[8];
            lds_children(t, d, i, gl, lane, lv[from], 0x0000FFFFu, v);
            const uint32_t w = meta_of(v);
            meta[((uint64_t)t.noff[d] + i) * m + c] = w;
            lv[from ^ 1][(i << gl) + lane] = w;
        }
    }
}

// Levels `from` .. 0 of the channels c_first .. of `chans`.
static ro_status meta_reduce(ro_octree *tr, int from, int gl, int c_first, uint32_t chans, hipStream_t s) {
    const TreeGeo &t = tr->t;
    const int m = tr->cache->vol->g.m, top = top_level(t, from);
    for (int d = from; d > top; --d) {
        hipLaunchKernelGGL(k_meta_reduce, dim3(nblocks(level_nodes(t, d) << gl)), dim3(256), 0, s, t, d,
                           tr->b.node_meta, m, gl, c_first, chans);
        RO_HIP(hipGetLastError());
    }
    if (top >= 0) {
        hipLaunchKernelGGL(k_meta_top, dim3(1), dim3(1024), 0, s, t, top, tr->b.node_meta, m, gl, c_first, chans);
        RO_HIP(hipGetLastError());
    }
    return RO_OK;
}

// The item that work index w (the same in the whole wave) belongs to: the
// last with start <= w.  The lanes probe 64 items at a time.
template <typename Item>
__device__ inline uint32_t find_item(const Item *__restrict__ items, uint32_t n_items, uint32_t w) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t lo = 0, hi = n_items;
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + 63) / 64, at = lo + lane * step;
        const uint32_t k = (uint32_t)__popcll(__ballot(at < hi && items[at].start <= w));  // lane 0 always
        lo += (k - 1) * step;
        hi = min(lo + step, hi);
    }
    return lo;
}

// Work item of the metadata-from-bricks pass: the leaves inside one
// resident brick (leaf grid coordinates, clipped to the grid).
struct MetaItem {
    uint32_t c, l, slot, b[3], x0, y0, z0, nx, ny, nz, start;  // start = prefix of leaf counts
};

// One wave per leaf: [min, max] over the voxels of the brick's level that
// overlap the leaf box dilated by one voxel of that level, clamped to the
// level's grid (at level 0: the L0 voxels within one voxel of the leaf).
// The dilated box stays inside the slot: the leaf lies inside the brick and
// the slot holds a one-voxel halo.  A box that misses the grid gives [0, 0].
__global__ __launch_bounds__(256) void k_meta_from_bricks(VolGeo g, TreeGeo t, const MetaItem *__restrict__ items,
                                                          uint32_t n_items, uint32_t w0, uint32_t n_work,
                                                          const uint8_t *__restrict__ slots,
                                                          uint32_t *__restrict__ meta,
                                                          uint8_t *__restrict__ level) {
    const uint32_t w = w0 + blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (w >= n_work) return;  // whole waves leave together
    const MetaItem it = items[find_item(items, n_items, w)];
    const uint32_t r = w - it.start;
    const uint32_t leaf[3] = {it.x0 + r % it.nx, it.y0 + (r / it.nx) % it.ny, it.z0 + r / (it.nx * it.ny)};
    const int l = (int)it.l;
    // metadata from finer data stay (the whole wave leaves together)
    const uint64_t li = ((((uint64_t)leaf[2] << t.nlog[t.depth][1]) + leaf[1]) << t.nlog[t.depth][0]) + leaf[0];
    uint8_t *lev = level + li * (uint64_t)g.m + it.c;
    if (*lev < (uint8_t)l) return;
    int vlo[3], vn[3];
    bool empty = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t x0 = (int64_t)leaf[a] << t.leaf_log[a];
        const int64_t x1 = x0 + (1ll << t.leaf_log[a]);
        const int sh = g.lshift[l][a];
        const int64_t a0 = (x0 >> sh) > 0 ? (x0 >> sh) - 1 : 0;
        const int64_t e = ((x1 - 1) >> sh) + 1, top = (int64_t)g.ldims[l][a] - 1;
        const int64_t a1 = e < top ? e : top;
        if (a0 > a1) empty = true;
        // slot coordinate of level voxel v: v - b * B + 1
        vlo[a] = (int)(a0 - ((int64_t)it.b[a] << g.Blog) + 1);
        vn[a] = (int)(a1 - a0 + 1);
    }
    uint32_t mn = 0xFFFFu, mx = 0;
    if (!empty) {
        const uint8_t *base = slots + (size_t)it.slot * g.slot_stride;
        const uint32_t E = (uint32_t)g.E;
        const int n = vn[0] * vn[1] * vn[2];
        // lane's voxel and the step of 64 voxels in (x, y, z) of the box, so
        // that a step is additions with carry in place of divisions; four
        // loads are in flight
        int x = lane % vn[0], y = (lane / vn[0]) % vn[1], z = lane / (vn[0] * vn[1]);
        const int sx = 64 % vn[0], sy = (64 / vn[0]) % vn[1], sz = 64 / (vn[0] * vn[1]);
        const uint32_t o0 = ((uint32_t)vlo[2] * E + (uint32_t)vlo[1]) * E + (uint32_t)vlo[0];
        for (int i = lane; i < n; i += 256) {
            uint32_t v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t o = o0 + ((uint32_t)z * E + (uint32_t)y) * E + (uint32_t)x;
                if (k == 0 || i + 64 * k < n)
                    v[k] = g.bpv == 1 ? (uint32_t)base[o] : (uint32_t)((const uint16_t *)base)[o];
                else v[k] = v[0];
                x += sx;
                const bool cx = x >= vn[0];
                x -= cx ? vn[0] : 0;
                y += sy + (cx ? 1 : 0);
                const bool cy = y >= vn[1];
                y -= cy ? vn[1] : 0;
                z += sz + (cy ? 1 : 0);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                mn = min(mn, v[k]);
                mx = max(mx, v[k]);
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            mn = min(mn, (uint32_t)__shfl_xor((int)mn, off));
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
        }
    } else {
        mn = 0;
    }
    if (lane == 0) {
        meta[(uint64_t)node_index(t, t.depth, leaf[0], leaf[1], leaf[2]) * g.m + it.c] = mn | (mx << 16);
        *lev = (uint8_t)l;
    }
}

ro_status octree_set_meta(ro_octree *tr, uint32_t c, const uint16_t *leaf_mm, hipStream_t s) {
    const TreeGeo &t = tr->t;
    const VolGeo &g = tr->cache->vol->g;
    const int m = g.m;
    const uint32_t unknown_max = g.bpv == 1 ? 255u : 65535u;
    const bool wide = (uintptr_t)leaf_mm % 4 == 0;
    hipLaunchKernelGGL(k_meta_leaf, dim3(nblocks(t.n_leaves)), dim3(256), 0, s, leaf_mm, wide, tr->b.node_meta,
                       tr->b.leaf_level, t.n_leaves, t.noff[t.depth], m, (int)c, unknown_max);
    RO_HIP(hipGetLastError());
    if (t.depth > 0) {
        hipLaunchKernelGGL(k_meta_parent, dim3(nblocks(level_nodes(t, t.depth - 1))), dim3(256), 0, s, t, leaf_mm,
                           wide, tr->b.node_meta, m, (int)c, unknown_max);
        RO_HIP(hipGetLastError());
    }
    return meta_reduce(tr, t.depth - 2, 0, (int)c, 1u << c, s);
}

// Residency mask of channel c at a leaf: bit l is set iff the level-l brick
// containing the leaf exists and is resident (each leaf lies in exactly one
// brick per level, so partial and full mapping coincide at leaves).
__device__ inline uint16_t leaf_mask(const VolGeo &g, const TreeGeo &t, const uint32_t *__restrict__ pt, int c,
                                     uint32_t lx, uint32_t ly, uint32_t lz) {
    uint16_t m = 0;
    const uint32_t x = lx << t.leaf_log[0], y = ly << t.leaf_log[1], z = lz << t.leaf_log[2];
    for (int l0 = 0; l0 < g.L; l0 += 4) {  // four entries in flight
        uint32_t e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int l = l0 + k < g.L ? l0 + k : l0;
            const uint32_t bx = x >> (g.Blog + g.lshift[l][0]);
            const uint32_t by = y >> (g.Blog + g.lshift[l][1]);
            const uint32_t bz = z >> (g.Blog + g.lshift[l][2]);
            const bool in = l0 + k < g.L && bx < (uint32_t)g.nb[l][0] && by < (uint32_t)g.nb[l][1] &&
                            bz < (uint32_t)g.nb[l][2];
            e[k] = in ? pt[dense_index(g, c, l, bx, by, bz)] : kInvalid;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) m |= (uint16_t)((e[k] != kInvalid ? 1u : 0u) << (l0 + k & 15));
    }
    return m;
}

__device__ inline uint32_t parent_of(const TreeGeo &t, int d, uint32_t x, uint32_t y, uint32_t z) {
    return node_index(t, d - 1, x >> (t.nlog[d][0] - t.nlog[d - 1][0]), y >> (t.nlog[d][1] - t.nlog[d - 1][1]),
                      z >> (t.nlog[d][2] - t.nlog[d - 1][2]));
}

// Inserted or evicted bricks of one channel and level: each overlaps the same
// box of leaves, 2^lo[a] per axis, so a work index gives its brick and leaf by
// shifts and the host sends 4 bytes a brick and no list of work.
struct LeafRun {
    uint32_t start;   // first work index
    uint32_t first;   // first brick in the list
    uint32_t cl;      // channel << 8 | level
    uint8_t log[3];   // log2 of the brick's leaves per axis
    uint8_t pad;
};
static_assert(sizeof(LeafRun) == 16, "LeafRun layout");

__global__ __launch_bounds__(256) void k_res_leaf(VolGeo g, TreeGeo t, const LeafRun *__restrict__ runs,
                                                  uint32_t n_runs, const uint32_t *__restrict__ bricks,
                                                  uint32_t n_work, const uint32_t *__restrict__ pt,
                                                  uint16_t *__restrict__ mask, uint8_t *__restrict__ flags) {
    const uint32_t w = blockIdx.x * 256 + threadIdx.x, w0 = w & ~63u;
    if (w0 >= n_work) return;  // whole waves leave together
    uint32_t k = find_item(runs, n_runs, w0);
    if (w >= n_work) return;
    while (k + 1 < n_runs && runs[k + 1].start <= w) ++k;  // runs that begin inside the wave
    const LeafRun run = runs[k];
    const uint32_t c = run.cl >> 8, l = run.cl & 255u;
    const uint32_t r = w - run.start, lx = run.log[0], ly = lx + run.log[1], lz = ly + run.log[2];
    const uint32_t lin = bricks[run.first + (r >> lz)] - c * g.per_channel - g.loff[l];
    const uint32_t nx = (uint32_t)g.nb[l][0], ny = (uint32_t)g.nb[l][1];
    const uint32_t row = lin / nx, bx = lin - row * nx, bz = row / ny, by = row - bz * ny;
    const uint32_t x = (bx << run.log[0]) + (r & ((1u << lx) - 1));
    const uint32_t y = (by << run.log[1]) + (r >> lx & ((1u << run.log[1]) - 1));
    const uint32_t z = (bz << run.log[2]) + (r >> ly & ((1u << run.log[2]) - 1));
    const uint16_t nm = leaf_mask(g, t, pt, (int)c, x, y, z);
    const uint32_t node = node_index(t, t.depth, x, y, z);
    uint16_t *p = mask + (uint64_t)node * g.m + c;
    if (*p != nm) {
        *p = nm;
        if (t.depth > 0) flags[parent_of(t, t.depth, x, y, z)] = 1;
    }
}

// Residency masks of the children of node i of level d in channel c.
__device__ inline void res_load(const TreeGeo &t, int d, uint32_t i, uint32_t c, int m, const uint16_t *mask,
                                uint32_t v[8]) {
    uint32_t x, y, z, c0[3], cn[3];
    node_coords(t, d, i, &x, &y, &z);
    child_range(t, d, x, y, z, c0, cn);
    const uint32_t n = cn[0] * cn[1] * cn[2], lx = cn[0] >> 1, ly = lx + (cn[1] >> 1);
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)  // an axis of one child takes no bit of k
        v[k] = k < n ? (uint32_t)mask[(uint64_t)node_index(t, d + 1, c0[0] + (k & (cn[0] - 1)),
                                                           c0[1] + ((k >> lx) & (cn[1] - 1)), c0[2] + (k >> ly)) *
                                          m + c]
                     : 0u;
}

// The wave's nodes of level d from i0 on, kResRounds at a time per group of
// 2^gl lanes (a lane per channel): flagged nodes get the OR of their
// children; a change flags the parent.  A lane per node reads the flags, so
// that a stretch without flags costs one load, and the rounds' loads are all
// issued before the first is used.
constexpr uint32_t kResRounds = 4;
__device__ inline void res_wave(const TreeGeo &t, int d, uint32_t i0, int m, int gl, uint16_t *mask, uint8_t *flags,
                                bool all) {
    const uint32_t n = (uint32_t)level_nodes(t, d), lane = threadIdx.x & 63, per = 64u >> gl;
    bool mine = false;
    if (lane < per * kResRounds && i0 + lane < n) {
        mine = all || flags[t.noff[d] + i0 + lane];
        if (mine && !all) flags[t.noff[d] + i0 + lane] = 0;
    }
    const unsigned long long want = __ballot(mine);
    const uint32_t c = lane & ((1u << gl) - 1), sub = lane >> gl;
    if (want == 0) return;
    uint32_t v[kResRounds][8], own[kResRounds];
    bool on[kResRounds];
#pragma unroll
    for (uint32_t r = 0; r < kResRounds; ++r) {
        const uint32_t k = r * per + sub;
        on[r] = k < 64 && (want >> (k & 63) & 1) && c < (uint32_t)m;
        if (!on[r]) continue;
        res_load(t, d, i0 + k, c, m, mask, v[r]);
        own[r] = mask[((uint64_t)t.noff[d] + i0 + k) * m + c];
    }
#pragma unroll
    for (uint32_t r = 0; r < kResRounds; ++r) {
        if (!on[r]) continue;
        uint32_t o = 0;
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) o |= v[r][k];
        if (o == own[r]) continue;
        const uint32_t i = i0 + r * per + sub;
        mask[((uint64_t)t.noff[d] + i) * m + c] = (uint16_t)o;
        if (d > 0 && !all) {
            uint32_t x, y, z;
            node_coords(t, d, i, &x, &y, &z);
            flags[parent_of(t, d, x, y, z)] = 1;
        }
    }
}

// Nodes per wave: at most 64 (one flag per lane).
static __host__ __device__ inline uint32_t res_wave_nodes(int gl) {
    return (64u >> gl) * kResRounds < 64 ? (64u >> gl) * kResRounds : 64;
}

// One level.  One thread per node walked 16 channels of 8 children in turn,
// 19 us a level whatever its size; with a lane per channel it is one round
// trip a round.
__global__ __launch_bounds__(256) void k_res_prop(TreeGeo t, int d, int m, int gl, uint16_t *mask, uint8_t *flags,
                                                  int all) {
    const uint64_t i0 = ((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * res_wave_nodes(gl);
    if (i0 < level_nodes(t, d)) res_wave(t, d, (uint32_t)i0, m, gl, mask, flags, all != 0);
}

// Levels d, d - 1, .. 0 by one block, if a node of level d is flagged: all
// nodes of level d from memory, the levels above from LDS (a node that is not
// flagged gets the masks that it has).  Clears the levels' flags.
__global__ __launch_bounds__(1024) void k_res_top(TreeGeo t, int d, int m, int gl, uint16_t *mask, uint8_t *flags,
                                                  int all) {
    __shared__ uint16_t lv[2][kTopNodes * kMaxC];
    const uint32_t lane = threadIdx.x & ((1u << gl) - 1), step = 1024u >> gl;
    const uint32_t n0 = (uint32_t)level_nodes(t, d);
    const bool on = lane < (uint32_t)m;
    if (!all) {
        bool any = false;
        for (uint32_t i = threadIdx.x; i < t.noff[d + 1]; i += 1024)
            if (flags[i]) {
                flags[i] = 0;
                any = true;
            }
        if (!__syncthreads_or(any)) return;
    }
    for (uint32_t i0 = threadIdx.x >> gl; i0 < n0; i0 += 4 * step) {
        uint32_t v[4][8], own[4];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = i0 + r * step;
            if (!on || i >= n0) continue;
            res_load(t, d, i, lane, m, mask, v[r]);
            own[r] = mask[((uint64_t)t.noff[d] + i) * m + lane];
        }
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = i0 + r * step;
            if (!on || i >= n0) continue;
            uint32_t o = 0;
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) o |= v[r][k];
            if (o != own[r]) mask[((uint64_t)t.noff[d] + i) * m + lane] = (uint16_t)o;
            lv[0][(i << gl) + lane] = (uint16_t)o;
        }
    }
    int from = 0;
    for (--d; d >= 0; --d, from ^= 1) {
        __syncthreads();
        const uint32_t n = (uint32_t)level_nodes(t, d);
        for (uint32_t i = threadIdx.x >> gl; i < n; i += step) {
            if (!on) continue;
            uint32_t v[8], o = 0;
            lds_children(t, d, i, gl, lane, lv[from], 0u, v);
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) o |= v[k];
            mask[((uint64_t)t.noff[d] + i) * m + lane] = (uint16_t)o;
            lv[from ^ 1][(i << gl) + lane] = (uint16_t)o;
        }
    }
}

static ro_status res_propagate(ro_octree *tr, int all, hipStream_t s) {
    const TreeGeo &t = tr->t;
    const int m = tr->cache->vol->g.m, gl = lanes_log(m), top = top_level(t, t.depth - 1);
    for (int d = t.depth - 1; d > top; --d) {
        const uint64_t per = 4 * res_wave_nodes(gl);
        hipLaunchKernelGGL(k_res_prop, dim3((unsigned)((level_nodes(t, d) + per - 1) / per)), dim3(256), 0, s, t, d, m, gl,
                           tr->b.node_mask, tr->b.node_flags, all);
        RO_HIP(hipGetLastError());
    }
    if (top >= 0) {
        hipLaunchKernelGGL(k_res_top, dim3(1), dim3(1024), 0, s, t, top, m, gl, tr->b.node_mask, tr->b.node_flags,
                           all);
        RO_HIP(hipGetLastError());
    }
    return RO_OK;
}

__global__ void k_res_leaf_all(VolGeo g, TreeGeo t, const uint32_t *__restrict__ pt, uint16_t *__restrict__ mask) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= t.n_leaves) return;
    const int D = t.depth;
    const uint32_t x = (uint32_t)(i & ((1u << t.nlog[D][0]) - 1));
    const uint32_t y = (uint32_t)((i >> t.nlog[D][0]) & ((1u << t.nlog[D][1]) - 1));
    const uint32_t z = (uint32_t)(i >> (t.nlog[D][0] + t.nlog[D][1]));
    const uint32_t node = t.noff[D] + (uint32_t)i;
    for (int c = 0; c < g.m; ++c) mask[(uint64_t)node * g.m + c] = leaf_mask(g, t, pt, c, x, y, z);
}

ro_status octree_update(ro_octree *tr, const std::vector<uint32_t> &dirty, hipStream_t s) {
    if (dirty.empty()) return RO_OK;
    const VolGeo &g = tr->cache->vol->g;
    const TreeGeo &t = tr->t;
    const int D = t.depth;
    // runs first, then the bricks, in the tree's scratch (its end is
    // the frame kernel's)
    constexpr size_t kRunBytes = 4096;
    constexpr size_t kRunsMax = kRunBytes / sizeof(LeafRun);  // as many channels x levels as a volume has
    const size_t cap = (tr->scratch_bytes - kFrameTail - kRunBytes) / sizeof(uint32_t);
    std::vector<LeafRun> runs;
    runs.reserve(kRunsMax);
    size_t first = 0, n_items = 0;  // bricks of the pending launch: dirty[first .. first + n_items)
    uint64_t work = 0;
    auto launch = [&]() -> ro_status {
        if (n_items == 0) return RO_OK;
        // one copy: the runs (a few), padded, and the bricks
        const size_t at = runs.size() * sizeof(LeafRun);
        uint8_t *list = nullptr;
        ro_status st = tr->list.make(at + n_items * sizeof(uint32_t), s, &list);
        if (st) return st;
        memcpy(list, runs.data(), at);
        memcpy(list + at, dirty.data() + first, n_items * sizeof(uint32_t));
        if ((st = tr->list.send(tr->b.scratch))) return st;
        hipLaunchKernelGGL(k_res_leaf, dim3(nblocks(work)), dim3(256), 0, s, g, t, (const LeafRun *)tr->b.scratch,
                           (uint32_t)runs.size(), (const uint32_t *)((uint8_t *)tr->b.scratch + at), (uint32_t)work,
                           tr->cache->b.page_table, tr->b.node_mask, tr->b.node_flags);
        RO_HIP(hipGetLastError());
        return RO_OK;
    };
    // The bricks are in ascending order, so those of one channel and level are
    // one run.  A brick's leaves: it starts at a multiple of its own edge
    // (a power of two of leaves), inside the leaf grid (another power of two).
    uint32_t run_end = 0;  // dense index where the current run's channel and level end
    uint32_t lz = 0;
    for (size_t i = 0; i < dirty.size(); ++i) {
        const uint32_t dn = dirty[i];
        const uint64_t cnt = 1ull << lz;
        const bool flush = n_items == cap || work + cnt > 0x7FFFFFFFull;
        if (flush || dn >= run_end) {
            const uint32_t c = dn / g.per_channel, r = dn - c * g.per_channel;
            int l = 0;
            while (l + 1 < g.L && g.loff[l + 1] <= r) ++l;
            LeafRun run = {};
            run.cl = c << 8 | (uint32_t)l;
            lz = 0;
            for (int a = 0; a < 3; ++a) {
                const int sh = g.Blog + g.lshift[l][a] - t.leaf_log[a];  // >= 0: leaf divides B
                run.log[a] = (uint8_t)std::min(sh, t.nlog[D][a]);
                lz += run.log[a];
            }
            run_end = c * g.per_channel + (l + 1 < g.L ? g.loff[l + 1] : g.per_channel);
            if (n_items == cap || work + (1ull << lz) > 0x7FFFFFFFull) {
                ro_status st = launch();
                if (st) return st;
                runs.clear();
                first = i;
                n_items = 0;
                work = 0;
            }
            run.start = (uint32_t)work;
            run.first = (uint32_t)n_items;
            runs.push_back(run);
        }
        ++n_items;
        work += 1ull << lz;
    }
    ro_status st = launch();
    if (!st) st = res_propagate(tr, 0, s);
    tr->list.mark();
    return st;
}

ro_status octree_rebuild(ro_octree *tr, hipStream_t s) {
    const VolGeo &g = tr->cache->vol->g;
    const TreeGeo &t = tr->t;
    hipLaunchKernelGGL(k_res_leaf_all, dim3(nblocks(t.n_leaves)), dim3(256), 0, s, g, t, tr->cache->b.page_table,
                       tr->b.node_mask);
    RO_HIP(hipGetLastError());
    ro_status st = res_propagate(tr, 1, s);
    if (st) return st;
    return launch_fill_u8(tr->b.node_flags, t.n_nodes, 0, s);
}


// Leaf metadata of the leaves inside resident bricks, computed from the
// bricks' voxels (Sec. 5.3, metadata on the client when the server has
// none).  `dense` holds validated resident dense indices sorted by level,
// coarsest first, so that where bricks of several levels cover one leaf the
// finest level's pass runs last and its values stay; a leaf whose metadata
// came from finer data (its level entry) keeps them.
ro_status octree_meta_from_bricks(ro_octree *tr, const std::vector<uint32_t> &dense, hipStream_t s) {
    if (dense.empty()) return RO_OK;
    const VolGeo &g = tr->cache->vol->g;
    const TreeGeo &t = tr->t;
    const int D = t.depth;
    const size_t cap = (tr->scratch_bytes - kFrameTail) / sizeof(MetaItem);
    // A level's items are one launch (the launches of coarser levels finish
    // first); all levels' items go up in one copy, and `start` counts anew in
    // each level.
    struct Run {
        size_t first;
        uint64_t work;
    };
    std::vector<MetaItem> items;
    std::vector<Run> runs;
    items.reserve(std::min(cap, dense.size()));
    runs.reserve(kMaxL);
    uint32_t chans = 0;
    int cur_level = -1;
    auto launch = [&]() -> ro_status {
        if (items.empty()) return RO_OK;
        uint8_t *list = nullptr;
        ro_status st = tr->list.make(items.size() * sizeof(MetaItem), s, &list);
        if (st) return st;
        memcpy(list, items.data(), items.size() * sizeof(MetaItem));
        if ((st = tr->list.send(tr->b.scratch))) return st;
        // at most 2^22 blocks of four waves per launch
        constexpr uint64_t kChunk = 1ull << 24;
        for (size_t k = 0; k < runs.size(); ++k) {
            const size_t end = k + 1 < runs.size() ? runs[k + 1].first : items.size();
            for (uint64_t w0 = 0; w0 < runs[k].work; w0 += kChunk) {
                const uint64_t nw = std::min(kChunk, runs[k].work - w0);
                hipLaunchKernelGGL(k_meta_from_bricks, dim3((unsigned)((nw + 3) / 4)), dim3(256), 0, s, g, t,
                                   (const MetaItem *)tr->b.scratch + runs[k].first, (uint32_t)(end - runs[k].first),
                                   (uint32_t)w0, (uint32_t)runs[k].work, (const uint8_t *)tr->cache->b.slots,
                                   tr->b.node_meta, tr->b.leaf_level);
                RO_HIP(hipGetLastError());
            }
        }
        return RO_OK;
    };
    for (uint32_t dn : dense) {
        const uint32_t c = dn / g.per_channel;
        const uint32_t r = dn - c * g.per_channel;
        int l = 0;
        while (l + 1 < g.L && g.loff[l + 1] <= r) ++l;
        const uint32_t lin = r - g.loff[l];
        const uint32_t b[3] = {lin % (uint32_t)g.nb[l][0], (lin / (uint32_t)g.nb[l][0]) % (uint32_t)g.nb[l][1],
                               lin / ((uint32_t)g.nb[l][0] * (uint32_t)g.nb[l][1])};
        MetaItem it;
        it.c = c;
        it.l = (uint32_t)l;
        it.slot = tr->cache->pt_host[dn];
        uint32_t lo[3], n[3];
        for (int a = 0; a < 3; ++a) {
            it.b[a] = b[a];
            const int sh = g.Blog + g.lshift[l][a] - t.leaf_log[a];  // >= 0: leaf divides B
            const uint64_t nl = 1ull << t.nlog[D][a];
            const uint64_t l0 = (uint64_t)b[a] << sh, l1 = std::min<uint64_t>(((uint64_t)b[a] + 1) << sh, nl);
            lo[a] = (uint32_t)std::min<uint64_t>(l0, nl);
            n[a] = l1 > l0 ? (uint32_t)(l1 - l0) : 0;
        }
        const uint64_t cnt = (uint64_t)n[0] * n[1] * n[2];
        if (cnt == 0) continue;
        if (items.size() == cap) {
            ro_status st = launch();
            if (st) return st;
            items.clear();
            runs.clear();
        }
        if (runs.empty() || l != cur_level || runs.back().work + cnt > 0x7FFFFFFFull) runs.push_back({items.size(), 0});
        cur_level = l;
        it.x0 = lo[0];
        it.y0 = lo[1];
        it.z0 = lo[2];
        it.nx = n[0];
        it.ny = n[1];
        it.nz = n[2];
        it.start = (uint32_t)runs.back().work;
        items.push_back(it);
        runs.back().work += cnt;
        chans |= 1u << c;
    }
    ro_status st = launch();
    if (!st) st = meta_reduce(tr, D - 1, lanes_log(g.m), 0, chans, s);
    tr->list.mark();
    return st;
}

}  // namespace ro
