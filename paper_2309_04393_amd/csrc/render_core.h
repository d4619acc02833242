// Per-ray core of the residency-octree ray caster, shared by the frame kernel
// (render.hip) and the multi-request serving kernel (serve.hip).
#pragma once

#include <math.h>

#include <type_traits>

#include "common.h"

namespace ro {

struct RenderArgs {
    // scalars
    int32_t dims[3];
    double sp[3];
    int32_t m, L, Blog, E, depth, start_level;
    uint32_t per_channel, slot_stride;
    double eye[3], F[3], R[3], U[3];
    double tx, ty, step, inv_step;
    int32_t proj, W, H;
    int32_t nvis;
    float term;
    uint32_t frame, flags;
    float win_k, win_0;  // a pixel's footprint in samples: win_0 + win_k * sample index
    int32_t ident;  // visible slot j shows channel j for every channel, and m % 4 == 0
    int32_t uni;    // every visible channel has the same level range (lo[0], hi[0])
    int32_t step_lo, step_hi;  // adaptive step: the finest desired level is clamped to these
    // uniform tables copied to LDS by the workgroup
    int32_t vis[kMaxC], lo[kMaxC], hi[kMaxC];
    uint32_t W0[kMaxC], W1[kMaxC];
    float w0[kMaxC], iw[kMaxC];
    uint32_t lsh[kMaxL];   // per level: packed log2 factors x | y << 8 | z << 16
    uint32_t loff[kMaxL];  // brick offset of the level inside a channel
    uint32_t nbx[kMaxL], nby[kMaxL];
    uint32_t K[kMaxL];     // level l is desired from sample index K[l] on
    uint32_t dd[kMaxL];    // traversal depth for the step of level l (the tree depth without the option)
    uint32_t nsh[kMaxD + 1];   // per tree level: packed log2 node edge
    uint32_t nlg[kMaxD + 1];   // per tree level: packed log2 node count
    uint32_t noff[kMaxD + 1];  // node offset of the level
    // device buffers
    const uint8_t *slots;
    const uint32_t *pt;
    uint32_t *cnt;
    uint32_t *stamp;
    const uint32_t *meta;
    const uint16_t *mask;
    const float4 *tf;
    float *rgba;
    uint32_t *aov;   // per-level reads (AOV kernel), or null
    uint32_t *reqb;  // required bricks per pixel, [H][W][1 + nvis] (AOV kernel), or null
    uint8_t *nodes;  // nodes whose metadata the frame reads, [n_nodes] (AOV kernel), or null
    unsigned long long *stats;
};

struct ChanLds {
    int c, lo, hi, nruns;
    uint32_t ehi;     // one zero-opacity run starting at raw value 0: its last raw value, else ~0
    uint32_t single;  // same in every entry: every visible channel has such a run
    uint32_t onecol;  // same in every entry: every visible channel's table has one colour
};

// Window and, where its table has one colour (onecol), colour of each visible
// channel, one row per value so that a group's values are one vector read.
// ehi: where every visible channel has one zero-opacity run starting at raw
// value 0, that run's last raw value in the upper half-word (a channel is
// empty in a node iff its metadata word does not exceed ehi | 0xFFFF); cbase:
// first brick of the channel.
// ax: what the set-up of a ray takes per axis.
struct AxisLds {
    double eye, F, R, U, sp, dim;
};
template <int NV>
struct __attribute__((aligned(16))) ChanPar {
    float w0[NV], iw[NV], r[NV], g[NV], b[NV];
    uint32_t ehi[NV], cbase[NV];
    AxisLds ax[3];
};

struct LevLds {
    uint32_t sh;   // packed shifts (level factor + brick) per axis
    uint32_t raw;  // packed level factor shifts
    uint32_t loff, nbx, nbxy, K;
    uint32_t dd;   // decision depth when this level sets the step
};

struct NodeLds {
    uint32_t nsh, nlg, noff;
};

__device__ __forceinline__ uint32_t field(uint32_t p, int a) { return (p >> (8 * a)) & 255u; }

// A pointer into device memory, marked as such: accesses through it are
// global (not flat) memory operations also where the frame's arguments were
// read from LDS (the serve kernels), where the compiler cannot tell.  The
// address goes through an integer: a cast to the global address space and
// straight back would be folded away.
template <class T>
__device__ __forceinline__ T *gmem(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)reinterpret_cast<uintptr_t>(p);
}

// Zero-alpha runs of a channel's table as raw-value bounds (lo | hi << 16):
// the range [mn, mx] is empty iff some run has mn >= lo and mx <= hi.  Raw
// values are at most 65535, so runs whose lower bound exceeds that are
// dropped and upper bounds are clamped to 65535.  Bounds from the window
// (24.8 fixed point, den = W1 - W0):
// floor(255 (256 r - W0) / den) >= a  <=>  r >= ceil((255 W0 + a den) / 65280)
// ceil (255 (256 r - W0) / den) <= b  <=>  r <= floor((255 W0 + b den) / 65280)
// zero: the entries of alpha 0, one bit each.
__device__ inline int build_runs(const uint64_t zero[4], uint32_t W0, uint32_t W1, uint32_t *runs) {
    int n = 0;
    const uint64_t den = (uint64_t)W1 - (uint64_t)W0;
    uint64_t prev = 0, w = zero[0], up = zero[1];  // the word before, at and after the scanned one
    int start = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        // entries at which a run starts or ends
        uint64_t first = w & ~((w << 1) | (prev >> 63)), last = w & ~((w >> 1) | (up << 63));
        while (first | last) {
            const int f = first ? __builtin_ctzll(first) : 64, l = last ? __builtin_ctzll(last) : 64;
            if (f <= l) {
                start = 64 * q + f;
                first &= first - 1;
                if (f != l) continue;
            }
            last &= last - 1;
            const int a = start, b = 64 * q + l;
            uint64_t rlo = a == 0 ? 0 : (255ull * W0 + (uint64_t)a * den + 65279ull) / 65280ull;
            uint64_t rhi = b == 255 ? 65535ull : (255ull * W0 + (uint64_t)b * den) / 65280ull;
            if (rhi > 65535ull) rhi = 65535ull;
            if (rlo <= rhi && n < kMaxRuns) runs[n++] = (uint32_t)rlo | ((uint32_t)rhi << 16);
        }
        prev = w;
        w = up;
        up = q == 0 ? zero[2] : q == 1 ? zero[3] : 0ull;
    }
    return n;
}

__device__ __forceinline__ bool range_empty(uint32_t mm, const uint32_t *runs, int nr) {
    const uint32_t mn = mm & 0xFFFFu, mx = mm >> 16;
    for (int r = 0; r < nr; ++r) {
        const uint32_t q = runs[r];
        if (mn >= (q & 0xFFFFu) && mx <= (q >> 16)) return true;
    }
    return false;
}

// A channel's transfer-function table in LDS: its 256 entries and a copy of
// the last, so the interpolation's upper entry needs no clamp.
constexpr int kTfStride = 257;

// Table position of raw value v in the window (w0, iw): entry (0 .. 255) and
// the weight of the next one.
__device__ __forceinline__ int tf_entry(float v, float w0, float iw, float &f) {
    float x = (v - w0) * iw;
    x = fminf(fmaxf(x, 0.0f), 1.0f);
    const int e = (int)(x * 255.0f);
    f = fmaf(x, 255.0f, -(float)e);
    return e;
}

// Two horizontally adjacent voxels (x, x + 1) in one load; the voxel grid
// is only 1- or 2-byte aligned, which global loads allow on this target.
template <int BPV>
__device__ __forceinline__ uint32_t vpair(const uint8_t *p) {
    if (BPV == 1) {
        uint16_t v;
        __builtin_memcpy(&v, p, 2);
        return v;
    }
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}

template <int BPV>
__device__ __forceinline__ void unpack(uint32_t w, float v[2]) {
    if (BPV == 1) {
        v[0] = (float)(w & 0xFFu);
        v[1] = (float)((w >> 8) & 0xFFu);
    } else {
        v[0] = (float)(w & 0xFFFFu);
        v[1] = (float)(w >> 16);
    }
}

__device__ __forceinline__ uint32_t brick_dense(const LevLds &lv, uint32_t c, uint32_t per_channel, int bx,
                                                int by, int bz) {
    return c * per_channel + lv.loff + (uint32_t)bz * lv.nbxy + (uint32_t)by * lv.nbx + (uint32_t)bx;
}

__device__ __forceinline__ uint32_t node_at(const NodeLds &nd, int x, int y, int z) {
    return nd.noff + ((((uint32_t)z << field(nd.nlg, 1)) + (uint32_t)y) << field(nd.nlg, 0)) + (uint32_t)x;
}

// Lanes per workgroup of the render and serve kernels.
#ifndef RO_LANES
#define RO_LANES 768
#endif
#ifndef RO_GROUP
#define RO_GROUP 4
#endif
constexpr int kRenderLanes = RO_LANES;
// Serving work items: up to kSegBlocks 8 x 8-pixel blocks of one request.
constexpr uint32_t kSegBlocks = 96;

// Channels whose loads are in flight together.
constexpr int group_of(int nv) { return nv < RO_GROUP ? nv : RO_GROUP; }

// Dynamic LDS of a workgroup: NV transfer-function tables, two entries of
// zeros (where the channels that are not sampled look up), then one slot word
// per ray and visible channel, the reciprocals of the ray directions, and
// each wave's table of miss counts.  P lanes work on a ray.
constexpr int kMissEntries = 32;
__host__ __device__ constexpr size_t render_lds_bytes(int nv, int p) {
    return ((size_t)nv * kTfStride + 2) * 16 + ((size_t)nv * 4 + 3 * 8) * (kRenderLanes / p) +
           (size_t)kMissEntries * 12 * (kRenderLanes / 64);
}

template <int G, class T>
__device__ __forceinline__ void group_read(const T *p, T v[G]) {
    if constexpr (G % 4 == 0) {
        typedef T vec4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int i = 0; i < G; i += 4) {
            const vec4 q = *(const vec4 *)(p + i);
            v[i] = q.x;
            v[i + 1] = q.y;
            v[i + 2] = q.z;
            v[i + 3] = q.w;
        }
    } else {
        for (int i = 0; i < G; ++i) v[i] = p[i];
    }
}

// A ray's LDS words: each visible channel's slot of the current visit (0 for
// a channel without one), kept in LDS rather than in registers, group-major
// so that a group's words are one vector read; and 1 / d.
template <int NV, int P>
struct RayLds {
    static constexpr int G = group_of(NV), kRays = kRenderLanes / P;
    uint32_t *p;  // this lane's words of the first group
    double *inv;  // this lane's first reciprocal
    uint32_t *miss;  // this wave's miss counts: key, channels (0: none), samples
    __device__ __forceinline__ RayLds(const float4 *s_tf) {
        uint32_t *w = (uint32_t *)(s_tf + kTfStride * NV + 2);
        p = w + threadIdx.x / P * G;
        inv = (double *)(w + NV * kRays) + threadIdx.x / P;
        miss = w + (NV + 6) * kRays + (threadIdx.x >> 6) * (3 * kMissEntries);
    }
    __device__ __forceinline__ uint32_t &slot(int j) { return p[(uint32_t)(j / G) * (kRays * G) + j % G]; }
    __device__ __forceinline__ void group(int g, uint32_t w[G]) const {
        group_read<G>(p + (uint32_t)(g / G) * (kRays * G), w);
    }
    __device__ __forceinline__ double &inverse(int a) { return inv[a * kRays]; }
};

// Pixel source of the stepping loop: a wave takes a unit of 64 / P pixels (8 x
// 8 for P = 1, 4 x 4 for P = 4) and the next one when all its rays have ended.
//
// Units of pixels are handed out by device counters (the units of an 8 x 8
// block, the blocks of a 32 x 32 tile are consecutive, tiles in raster
// order).  With n_queues = 1 one counter hands out the units in order.  With
// n_queues > 1 they are dealt in chunks of `chunk` consecutive units, chunk c
// to queue c mod n_queues; a workgroup starts on queue (workgroup index mod
// n_queues), which with workgroups dealt to the XCDs in turn is its XCD's,
// and takes from the next queues once its own is used up; the wave that finds
// a queue used up tells the workgroup's others in LDS.  In large frames a
// workgroup takes a few units at once and its waves share them.  The XCDs then
// work on separate neighbouring chunks (their L2s hold different lines)
// while all of them still sweep the image together (the Infinity Cache is
// shared).  Counter reads and the unit are wave-uniform.
//
// Per-XCD block queues: blocks are dealt to them in chunks of RO_CHUNK
// consecutive blocks (16 chunks per queue at 1080p).  On the 16-channel
// 1080p frame chunks of 256 measured 0.6 % faster than 64, 16 0.7 % slower,
// 1024 as 256, and 4096 (one region per XCD) 4 % slower (with one lane per ray).
#ifndef RO_QUEUES
#define RO_QUEUES 8
#endif
#ifndef RO_CHUNK
#define RO_CHUNK 256
#endif
// Words between queue counters: 256 bytes, so that they are in different
// memory channels.  At 32 bytes a 1080p frame of short rays with an atomic
// per unit waited for the atomics of one channel (homogeneous nodes 0.84 ms,
// 0.39 at 256; with several units per atomic 0.37 and 0.35).
constexpr int kQueueStride = 64;
// Units that a workgroup takes at once, by the units that the image has per
// wave.  One atomic for several units leaves the queues' memory channels alone
// (1080p with nothing in view: 0.30 ms with one, 0.24 with two, 0.15 with
// four), and neighbouring waves work on neighbouring pixels (4 channels far
// away 1.20, 0.99, 0.95; a batch of twelve requests 51.8, 44.8, 44.8; a
// fly-through of 16 channels 84.3, 84.0, 83.4, though the fabric brings 124,
// 143, 166 GB a frame).  But the frame waits for the workgroup whose units are the heavy ones: far away
// 1.29 with eight; 720p, 8 channels, 19 units a wave: 3.28, 3.28, 3.35; 512 x
// 512, 5 units a wave: 2.10 with one, 2.25 with four.
constexpr uint32_t kMaxTake = 4;
__host__ __device__ inline uint32_t units_at_once(uint32_t n_units, uint32_t waves) {
    return n_units >= 32 * waves ? kMaxTake : n_units >= 8 * waves ? 2 : 1;
}
static_assert(RO_QUEUES * kQueueStride * 4 <= kFrameTail, "unit counters");
// Blocks per chunk of an image of n_blocks: smaller images in smaller chunks,
// whole 32 x 32 tiles of them.
__host__ __device__ inline uint32_t queue_chunk(uint32_t n_blocks) {
    const uint32_t c = n_blocks / (RO_QUEUES * 8);
    return c >= RO_CHUNK ? RO_CHUNK : c >= 16 ? c & ~15u : c ? c : 1;
}

// A workgroup's share of the unit queues (LDS).
struct UnitLds {
    uint32_t used;  // queues found used up, a bit each
    uint32_t lock;  // a wave is taking the next batch
    unsigned long long batch;  // first unit << 32 | units of the batch handed out
    __device__ __forceinline__ void clear() {
        used = lock = 0;
        batch = 0x7FFFFFFFull;  // none left
    }
};

template <int P>
struct UnitQueue {
    uint32_t *counter;  // n_queues counters kQueueStride words apart, zero at launch (device or LDS)
    uint32_t n_units;   // units this queue hands out: offset .. offset + n_units - 1
    uint32_t offset, tiles_x;
    uint32_t n_queues, chunk;
    uint32_t split;     // log2 of the parts that a unit's pixels are handed out in (P = 4 only)
    uint32_t take;      // units that a workgroup takes at once (1, 2 or 4; chunk is a multiple of 4 where not 1)
    UnitLds *wg;        // cleared at the start
    int W, H;
    bool exhausted;
    uint32_t q;         // current queue (wave-uniform)
    uint32_t taken;     // units handed out to this wave

    __device__ __forceinline__ void init() {
        q = blockIdx.x % n_queues;
        taken = 0;
        exhausted = false;
    }
    // First of the next `take` units of a queue that is not used up, or n_units.
    __device__ __forceinline__ uint32_t pop_queue() {
        // (each turn takes units, goes on to a queue that is not used up, or marks one that is)
        uint32_t seen;
        while ((seen = __hip_atomic_load(&wg->used, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) !=
               (1u << n_queues) - 1) {
            if (seen >> q & 1u) {
                q = (q + 1) % n_queues;
                continue;
            }
            const uint32_t i = atomicAdd(counter + q * kQueueStride, take);
            const uint64_t u = ((uint64_t)(i / chunk) * n_queues + q) * chunk + i % chunk;
            if (u < n_units) return (uint32_t)u;
            __hip_atomic_fetch_or(&wg->used, 1u << q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        return n_units;
    }
    // Next unit of the workgroup's batch; the wave that finds none left takes
    // the next batch while the others wait for it (it waits for nobody).
    __device__ __forceinline__ uint32_t pop_batch() {
        while (true) {
            const unsigned long long w =
                __hip_atomic_fetch_add(&wg->batch, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if ((uint32_t)w < take) {
                const uint32_t u = (uint32_t)(w >> 32) + (uint32_t)w;
                if (u < n_units) return u;
                continue;  // past the end of the last chunk
            }
            uint32_t free = 0;
            if (!__hip_atomic_compare_exchange_strong(&wg->lock, &free, 1u, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_WORKGROUP)) {
                __builtin_amdgcn_s_sleep(1);
                continue;
            }
            uint32_t u = 0;
            if ((uint32_t)__hip_atomic_load(&wg->batch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= take) {
                u = pop_queue();
                if (u < n_units)
                    __hip_atomic_store(&wg->batch, (unsigned long long)u << 32, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __hip_atomic_store(&wg->lock, 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (u >= n_units) return n_units;
        }
    }
    __device__ __forceinline__ uint32_t pop() {
        uint32_t b = n_units;
        if ((threadIdx.x & 63) == 0)
            b = n_queues == 1 ? atomicAdd(counter, 1u) : take == 1 ? pop_queue() : pop_batch();
        q = (uint32_t)__builtin_amdgcn_readfirstlane((int)q);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
    }
    // this lane's pixel of the next unit; false (in every lane) when there is none
    __device__ __forceinline__ bool next(int &x, int &y, bool &v) {
        if (exhausted) return false;
        uint32_t u = pop();
        if (u >= n_units) {
            exhausted = true;
            return false;
        }
        ++taken;
        u += offset;
        const uint32_t i = (threadIdx.x & 63u) / P, part = u & ((1u << split) - 1);
        u >>= split;
        const uint32_t b = u / P, t = b >> 4;
        x = (int)((t % tiles_x) * 32 + (b & 3u) * 8);
        y = (int)((t / tiles_x) * 32 + ((b >> 2) & 3u) * 8);
        if (P == 4) {
            // 2 x 2 pixels are neighbouring lanes: the 16 lanes whose gathers
            // are looked up together touch fewer cache lines than with rows
            // of four (18.5 against 22.5 lookups per 64-lane load)
            x += (int)((u & 1u) * 4 + (i & 1u) + (i >> 1 & 2u));
            y += (int)((u >> 1 & 1u) * 4 + (i >> 1 & 1u) + (i >> 2 & 2u));
        } else {
            x += (int)(i & 7u);
            y += (int)(i >> 3);
        }
        v = x < W && y < H && (P != 4 || (i >> (4 - split)) == part);
        return true;
    }
};

// Slot bytes of a brick of edge e (halo included): rounded up to 256 bytes,
// as the cache lays out its slots.
__host__ __device__ constexpr size_t slot_bytes(int e, int bpv) {
    return ((size_t)e * e * e * bpv + 255) / 256 * 256;
}

// A value that is the same in every lane (a kernel argument, or a field of
// the workgroup's staged request) as a scalar of its own: kept in scalar
// registers by itself instead of being read again with its neighbours.
__device__ __forceinline__ uint32_t scalar32(uint32_t x) {
    x = (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
    asm volatile("" : "+s"(x));
    return x;
}
__device__ __forceinline__ uint64_t scalar64(uint64_t x) {
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    uint64_t v = ((uint64_t)hi << 32) | (uint64_t)lo;
    asm volatile("" : "+s"(v));
    return v;
}

// The value of lane i of the P lanes of this lane's ray.
template <int P, int i>
__device__ __forceinline__ uint32_t ray_lane(uint32_t v) {
    if constexpr (P == 1) return v;
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, i * 0x55, 0xf, 0xf, true);  // quad_perm i i i i
}
template <int P, int i>
__device__ __forceinline__ float ray_lane(float v) {
    return __uint_as_float(ray_lane<P, i>(__float_as_uint(v)));
}
template <int P, int i>
__device__ __forceinline__ double ray_lane(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint64_t r = (uint64_t)ray_lane<P, i>((uint32_t)(b >> 32)) << 32 | ray_lane<P, i>((uint32_t)b);
    return __longlong_as_double((long long)r);
}

// Smallest of the wave's values, in every lane.
__device__ __forceinline__ float wave_min(float v) {
    // row_shr 1, 2, 4, 8 within rows of 16, then the row and half broadcasts: lane 63 holds the minimum
#define RO_STEP(ctrl)                                                                                        \
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), ctrl, 0xf, \
                                                            0xf, false)));
    RO_STEP(0x111)
    RO_STEP(0x112)
    RO_STEP(0x114)
    RO_STEP(0x118)
    RO_STEP(0x142)
    RO_STEP(0x143)
#undef RO_STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The lanes of a wave exchange values through LDS without a barrier of the
// workgroup (the miss table; the slot words of a ray): what lanes wrote before
// this point is what all lanes read after it, and what they read before it is
// what was there.  LDS serves a wave in order, so it costs no instruction; it
// keeps the compiler from taking a lane's last store or load for the word's
// value.  Called by the whole wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// EC: the brick edge with halo known at compile time (0: read from A).  A
// constant edge turns the four gather offsets into instruction immediates.
// EXT: bit 0 render-and-skip of nodes homogeneous for all channels, bit 1
// per-channel sampling rates (frames that ask for them go to a kernel that
// has them).
//
// A lane alternates between visits and samples.  A visit takes the ray's next
// sample position, descends to its leaf, skips an empty node, or finds the
// slot of each channel and the last sample that lies in the leaf (the visit's
// segment).  The samples of a segment then need no tree or level logic: the
// position, scaled to the level's voxels (an exact power of two), is one
// multiply-add per axis.
template <int NV, int BPV, bool AOV, int EC, int EXT, int P>
__device__ __forceinline__ void render_rays(const RenderArgs &A, UnitQueue<P> &src, const float4 *s_tf,
                                            const ChanLds *s_ch, const ChanPar<NV> *s_par, const uint32_t *s_runs,
                                            const LevLds *s_lv, const NodeLds *s_nd, uint32_t stats[7]) {
    constexpr bool HOMOG = (EXT & 1) != 0;
    constexpr bool RATES = (EXT & 2) != 0;
    const int nvis = (int)scalar32((uint32_t)A.nvis);
    const int D = (int)scalar32((uint32_t)A.depth);
    const int L = (int)scalar32((uint32_t)A.L);
    const int m = (int)scalar32((uint32_t)A.m);
    const double step = __longlong_as_double((long long)scalar64((uint64_t)__double_as_longlong(A.step)));
    const uint8_t *pool = (const uint8_t *)(const __attribute__((address_space(1))) uint8_t *)scalar64(
        reinterpret_cast<uint64_t>(A.slots));
    const bool onecol = scalar32(s_ch[0].onecol) != 0;
    constexpr int kGroup = group_of(NV);  // gathers
    // The P lanes of a ray share a visit's channels: lane q takes the kOwn
    // channels from q * kOwn on, vGroup at a time.
    constexpr int kOwn = NV > P ? NV / P : 1;
    constexpr int vGroup = kOwn < 4 ? kOwn : 4;
    const int q = P == 1 ? 0 : (int)(threadIdx.x & (P - 1));
    const int own = min(q * kOwn, NV - kOwn);  // (with more lanes than channels the last ones repeat a channel)
    // OR over the lanes of a ray
    auto all_of_ray = [&](uint32_t v) {
        if (P == 4) {
            v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, true);  // quad_perm 1 0 3 2
            v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, true);  // quad_perm 2 3 0 1
        }
        return v;
    };
    const double one_minus_term = 1.0 - (double)A.term;
    const uint32_t vismask = (nvis >= 32) ? 0xFFFFFFFFu : ((1u << nvis) - 1u);
    const int s0 = A.start_level;
    const bool noskip = (A.flags & RO_RENDER_NO_SKIP) != 0;
    const bool adaptive = (A.flags & RO_RENDER_ADAPTIVE_STEP) != 0;
    const bool homog = HOMOG && (A.flags & RO_RENDER_HOMOGENEOUS) != 0;
    // per-channel sampling rates (with the adaptive step): a channel takes part
    // only in samples k that are multiples of its own level's x factor
    const bool rates = RATES && adaptive && (A.flags & RO_RENDER_CHANNEL_RATES) != 0;
    // traversal depth from the step (with the adaptive step): emptiness and
    // homogeneity are decided at the node of depth dd of the step's level
    const bool tdepth = adaptive && (A.flags & RO_RENDER_TRAVERSAL_DEPTH) != 0;
    const bool per_sample = rates || (AOV && (A.aov || A.reqb));  // every sample is recorded by itself
    const NodeLds leafl = s_nd[D];
    const bool single = s_ch[0].single != 0;
    const float2 *s_tfa = (const float2 *)s_tf;
    RayLds<NV, P> lds(s_tf);
    const uint32_t E = EC ? (uint32_t)EC : (uint32_t)A.E;
    const uint32_t stride = EC ? (uint32_t)slot_bytes(EC, BPV) : A.slot_stride;
    uint32_t st_samples = 0, st_reads = 0, st_miss = 0, st_visits = 0, st_nonempty = 0, st_iters = 0, st_hom = 0;

    // ---- per-ray state
    int px = 0, py = 0;
    bool has = false;  // the lane holds a ray (finished or not)
    // ray in voxels of the level whose factors are 2^vsh (per axis; 0: L0)
    double o[3] = {0, 0, 0}, d[3] = {0, 0, 0};
    uint32_t vsh = 0;
    double Cr = 0, Cg = 0, Cb = 0, Tr = 1.0;
    float *out = nullptr;
    bool done = true;
    // sample index, last index of the ray, first index past the segment (whole numbers)
    double k = 0, kend = -1, kseg = 0;
    int rsh = 0;  // adaptive step: log2 of the segment's sampling distance
    uint32_t cur_leaf = kInvalid;
    int cur_lod = -1, lod = 0;
    double klod = INFINITY;  // first sample index of the next level
    uint32_t emask = 0, missmask = 0;
    uint64_t lvpack = 0;
    // samples not yet added to the miss counters: their count, the missing
    // channels, and the finest desired brick (x | y << 8 | z << 16) and
    // level index (<< 24) they share
    uint32_t npend = 0, pmask = 0, pkey = 0;
    uint32_t fpend = 0, fmask = 0, fkey = 0;  // those of the visit before, to be added
    uint32_t smiss = 0;            // with rates: this lane's sample's missing channels, to be added
    int lc[3] = {-1, -1, -1};      // L0 origin of the last visited leaf or skipped node (none yet)
    int lcd = 0;                   // its depth: the nodes above it are known not to be skipped
    uint32_t last_key = kInvalid;  // (level, cell) of the last visit when uniform
    uint32_t cbias = 0;            // when uniform: voxel index of the brick's origin in its level's slot strides
    uint32_t have = 0;             // channels with a slot from the last visit
    uint32_t stamped = 0;          // with rates: channels whose current slot carries this frame's stamp
    uint64_t rpk = 0;              // with rates: each channel's rate shift in the current visit (4 bits)

    auto next_level = [&]() {
        ++lod;
        const uint32_t K = lod + 1 < L ? s_lv[lod + 1].K : kInvalid;
        klod = K == kInvalid ? INFINITY : (double)K;
    };

    // ray set-up in L0 voxel units, box interval, first sample index; lane q
    // of a ray's four takes axis q (the last one repeats axis 2).  With every
    // lane taking every axis, and a phase of the wave for each sample before
    // the volume, it was a third of the instructions of rays that end at once
    // (1080p, 4 channels, 2.4 samples a pixel: 0.50 ms to 0.43)
    auto start = [&](int x, int y, bool valid) {
        px = x;
        py = y;
        has = true;
        constexpr int kAxes = P == 4 ? 1 : 3;  // of a lane
        // (taken from the lane anew, or its addresses would be kept through
        // the ray loop)
        uint32_t ln = threadIdx.x;
        asm volatile("" : "+v"(ln));
        const int q = P == 1 ? 0 : (int)(ln & (P - 1));
        const int a0 = P == 4 ? min(q, 2) : 0;
        // (fused multiply-adds are written out where positions and samples are
        // computed: which products the compiler fuses would otherwise depend
        // on the code around them)
        double a, b;
        {
            const int na = 2 * px + 1 - A.W, nb = A.H - 2 * py - 1;
            if constexpr (P == 4) {
                const double r = (double)(q & 1 ? nb : na) / (double)(q & 1 ? A.H : A.W);
                a = ray_lane<P, 0>(r);
                b = ray_lane<P, 1>(r);
            } else {
                a = (double)na / (double)A.W;
                b = (double)nb / (double)A.H;
            }
        }
        const double ax = a * A.tx, by = b * A.ty;
        double ow[kAxes], dw[kAxes], dim[kAxes];
        if (A.proj == RO_PROJ_ORTHO) {
#pragma unroll
            for (int i = 0; i < kAxes; ++i) {
                const AxisLds &X = s_par->ax[a0 + i];
                ow[i] = fma(by, X.U, fma(ax, X.R, X.eye));
                dw[i] = X.F;
            }
        } else {
#pragma unroll
            for (int i = 0; i < kAxes; ++i) {
                const AxisLds &X = s_par->ax[a0 + i];
                ow[i] = X.eye;
                dw[i] = fma(by, X.U, fma(ax, X.R, X.F));
            }
            const double w0 = ray_lane<P, 0>(dw[0]), w1 = ray_lane<P, 1>(dw[kAxes / 2]),
                         w2 = ray_lane<P, 2>(dw[kAxes - 1]);
            double n = fma(w2, w2, fma(w0, w0, w1 * w1));
            n = sqrt(n);
#pragma unroll
            for (int i = 0; i < kAxes; ++i) dw[i] = dw[i] / n;
        }
        double t0 = -INFINITY, t1 = INFINITY;
        uint32_t miss = valid ? 0u : 1u;
#pragma unroll
        for (int i = 0; i < kAxes; ++i) {
            const AxisLds &X = s_par->ax[a0 + i];
            dim[i] = X.dim;
            ow[i] = ow[i] / X.sp;
            dw[i] = dw[i] / X.sp;
            lds.inverse(a0 + i) = 1.0 / dw[i];
            if (dw[i] == 0.0) {
                if (ow[i] < 0.0 || ow[i] >= dim[i]) miss = 1;
                continue;
            }
            const double u = (0.0 - ow[i]) / dw[i], v = (dim[i] - ow[i]) / dw[i];
            t0 = fmax(t0, u > v ? v : u);
            t1 = fmin(t1, u > v ? u : v);
        }
        miss = all_of_ray(miss);
        if constexpr (P == 4) {
            t0 = fmax(fmax(ray_lane<P, 0>(t0), ray_lane<P, 1>(t0)), ray_lane<P, 2>(t0));
            t1 = fmin(fmin(ray_lane<P, 0>(t1), ray_lane<P, 1>(t1)), ray_lane<P, 2>(t1));
        }
        o[0] = ray_lane<P, 0>(ow[0]);
        o[1] = ray_lane<P, 1>(ow[kAxes / 2]);
        o[2] = ray_lane<P, 2>(ow[kAxes - 1]);
        d[0] = ray_lane<P, 0>(dw[0]);
        d[1] = ray_lane<P, 1>(dw[kAxes / 2]);
        d[2] = ray_lane<P, 2>(dw[kAxes - 1]);
        vsh = 0;
        Cr = Cg = Cb = 0.0;
        Tr = 1.0;
        out = valid ? gmem(A.rgba) + ((size_t)py * A.W + px) * 4 : nullptr;
        if (AOV && A.reqb && valid) {
            // required bricks: the count, then each channel's last desired brick
            uint32_t *rb = A.reqb + ((size_t)py * A.W + px) * (1 + nvis);
            rb[0] = 0;
            for (int j = 0; j < nvis; ++j) rb[1 + j] = kInvalid;
        }
        done = miss || t0 > t1;
        double k0, k1;
        if constexpr (P == 4) {
            const double r = (q & 1 ? t1 : t0) / A.step;
            k0 = ray_lane<P, 0>(r);
            k1 = ray_lane<P, 1>(r);
        } else {
            k0 = t0 / A.step;
            k1 = t1 / A.step;
        }
        k = done ? 0.0 : floor(k0) - 1.0;
        if (!(k > 0.0)) k = 0.0;
        kend = done ? -1.0 : ceil(k1) + 1.0;
        // a ray without an end inside the volume (a camera without a direction) has no samples
        if (!(kend < 9.0e15)) {
            done = true;
            kend = -1.0;
        }
        // on to the first sample inside the volume, one or two as a rule
        while (!done && k <= kend) {
            const double t = k * step;
            uint32_t outside = 0;
#pragma unroll
            for (int i = 0; i < kAxes; ++i) {
                const double u = fma(t, dw[i], ow[i]);
                outside |= u >= 0.0 && u < dim[i] ? 0u : 1u;
            }
            if (!all_of_ray(outside)) break;
            k += 1.0;
        }
        kseg = k;
        rsh = 0;
        cur_leaf = kInvalid;
        cur_lod = -1;
        lod = -1;
        klod = -1.0;
        while (k >= klod) next_level();
        emask = missmask = 0;
        lvpack = 0;
        npend = pmask = 0;
        lc[0] = lc[1] = lc[2] = -1;
        lcd = 0;
        last_key = kInvalid;
        have = 0;
        stamped = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) lds.slot(j) = 0;
    };

    // Adds n samples to the miss counters of the channels in msk at the
    // desired bricks of key: lane j the counter of channel j.
    auto count_misses = [&](uint32_t key, uint32_t msk, uint32_t n) {
        const int ln = (int)(threadIdx.x & 63u);
        if (ln < NV && ((msk >> ln) & 1u)) {
            const int plod = (int)(key >> 24);
            const LevLds lf = s_lv[min(max(plod, A.step_lo), A.step_hi)];
            const ChanLds ch = s_ch[ln];
            const LevLds lv = s_lv[min(max(plod, ch.lo), ch.hi)];
            // the desired brick is as coarse as the shared one or coarser and contains it
            const uint32_t s = lv.sh - lf.sh;
            atomicAdd(&gmem(A.cnt)[brick_dense(lv, (uint32_t)ch.c, A.per_channel, field(key, 0) >> field(s, 0),
                                               field(key, 1) >> field(s, 1), field(key, 2) >> field(s, 2))],
                      n);
        }
    };
    // Pending samples go to the miss counters by way of a table of the wave
    // (kMissEntries sums in LDS, by brick and missing channels).  Device
    // atomics leave the XCD, and on a frame with few bricks every ray of a
    // wave, and the next units' rays, add to the same counters: one atomic per
    // ray, visit and channel took 26 ms of a 960 x 540 frame of a 16-channel
    // slide without bricks, one per wave and brick 7.  (With rates the samples
    // of a ray differ in the channels that take part, so each is added by
    // itself: a 1080p frame of 8 channels, half of the bricks resident, 250 ms
    // with an atomic per sample and channel, 25 now.)
    // (Called by the whole wave: every lane takes part.)
    auto flush = [&](uint32_t n_own, uint32_t mask, uint32_t key_own) {
        uint64_t todo = __ballot(n_own != 0 && mask != 0);
        const int ln = (int)(threadIdx.x & 63u);
        while (todo) {
            const int first = __builtin_ctzll(todo);
            const uint32_t key = (uint32_t)__builtin_amdgcn_readlane((int)key_own, first);
            const uint32_t msk = (uint32_t)__builtin_amdgcn_readlane((int)mask, first);
            const bool mine = ((todo >> ln) & 1ull) && key_own == key && mask == msk;
            const uint64_t like = __ballot(mine);
            uint32_t n = mine ? n_own : 0u;
            st_miss += n * (uint32_t)__popc(msk);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
            uint32_t *e = lds.miss + 3 * ((((key ^ key >> 13) * 0x9E3779B1u) >> 16 ^ msk) % kMissEntries);
            const uint32_t ek = e[0], em = e[1], en = e[2];
            const bool hit = ek == key && em == msk;
            if (!hit && em) count_misses(ek, em, en);
            wave_sync();
            if (ln == 0) {
                e[0] = key;
                e[1] = msk;
                e[2] = hit ? en + n : n;
            }
            wave_sync();
            todo &= ~like;
        }
    };

    auto finish = [&]() {
        if (out && q == 0) *(float4 *)out = make_float4((float)Cr, (float)Cg, (float)Cb, (float)(1.0 - Tr));
        has = false;
        npend = 0;
    };

    // The next sample position of a ray: skip the node it lies in, or set up
    // the segment of its leaf.
    auto visit = [&]() {
        double oo[3], dd[3], u[3];
        const double t = k * step;
        bool inside = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int s = (int)field(vsh, a);
            oo[a] = ldexp(o[a], s);
            dd[a] = ldexp(d[a], s);
            u[a] = fma(t, dd[a], oo[a]);
            inside = inside && (u[a] >= 0.0) && (u[a] < (double)A.dims[a]);
        }
        if (!inside) {
            k += 1.0;
            kseg = k;
            return;
        }
        const int iu[3] = {(int)u[0], (int)u[1], (int)u[2]};
        while (k >= klod) next_level();
        // LOD-adaptive step: the finest desired level over the visible
        // channels sets the sampling distance, r = its x factor; only samples
        // with k a multiple of r are evaluated
        int dend = D;
        rsh = 0;
        if (adaptive) {
            const LevLds slv = s_lv[min(max(lod, A.step_lo), A.step_hi)];
            rsh = (int)field(slv.raw, 0);
            if (tdepth) dend = (int)slv.dd;
            const double up = ldexp(ceil(ldexp(k, -rsh)), rsh);
            if (up != k) {
                k = up;
                kseg = k;
                return;
            }
        }
        const uint32_t leaf = node_at(leafl, iu[0] >> field(leafl.nsh, 0), iu[1] >> field(leafl.nsh, 1),
                                      iu[2] >> field(leafl.nsh, 2));
        uint32_t end_nsh = leafl.nsh;  // node whose exit ends the segment
        bool skip = false;
        const bool same = leaf == cur_leaf && lod == cur_lod;
        uint32_t rs_node = 0, rs_mask = 0;  // render-and-skip: the node and its homogeneous channels
        // with a traversal depth the decision node depends on the level too
        if (leaf != cur_leaf || (tdepth && lod != cur_lod)) {
            // Descend from the start level and skip the first node that
            // is empty for every visible channel (the leaf included).
            // Every ancestor of a visited leaf is non-empty, so levels
            // whose node also holds the last visited leaf are known
            // non-empty and the test starts below them (the same node
            // is skipped either way).  With HOMOG the first node in which
            // every visible channel is empty or holds one value (and one
            // holds a value) is rendered from those values and skipped
            // (Alg. 1 renderAndSkipNode, Sec. 6.1: homogeneous for all
            // channels): its samples are composited and the ray goes on
            // past the node.  Ancestors of a visited leaf are never such
            // nodes either (metadata nest, so their descendants would be),
            // and the ancestors of a skipped node were tested and found
            // not to be skipped: the shared levels above the last visited
            // leaf or skipped node are not tested again.  An axis whose leaf
            // coordinates differ in their lowest n bits only is shared down to
            // depth D - n (an axis is split at the last of the levels).
            int d0 = noskip ? dend : min(s0, dend);
            if (lc[0] >= 0 && !noskip && !tdepth) {
                const uint32_t x = (uint32_t)(iu[0] ^ lc[0]) >> field(leafl.nsh, 0),
                               y = (uint32_t)(iu[1] ^ lc[1]) >> field(leafl.nsh, 1),
                               z = (uint32_t)(iu[2] ^ lc[2]) >> field(leafl.nsh, 2);
                const int n = 32 - __clz((int)(x | y | z));  // the longest of the three
                d0 = max(d0, min(lcd, D - n + 1));
            }
            for (int dl = d0; dl <= dend; ++dl) {
                const NodeLds nd = s_nd[dl];
                const uint32_t node = node_at(nd, iu[0] >> field(nd.nsh, 0), iu[1] >> field(nd.nsh, 1),
                                              iu[2] >> field(nd.nsh, 2));
                // the node's metadata, vGroup channels per batch of loads
                uint32_t em = 0, hm = 0;
                const uint32_t *nm = gmem(A.meta) + (size_t)node * m;
                if (AOV && A.nodes) A.nodes[node] = 1;
#pragma unroll
                for (int g = 0; g < kOwn; g += vGroup) {
                    const int j0 = own + g;
                    if (P == 1 && g >= nvis) break;
                    uint32_t mm[vGroup];
                    if (vGroup > 1 && A.ident) {
                        group_read<vGroup>(nm + min(j0, nvis - vGroup), mm);  // one aligned load
                    } else {
#pragma unroll
                        for (int jj = 0; jj < vGroup; ++jj) mm[jj] = nm[s_ch[j0 + jj].c];
                    }
                    if (single) {
                        // one zero run [0, ehi] per channel: empty iff the maximum is within it
                        uint32_t eh[vGroup];
                        group_read<vGroup>(s_par->ehi + j0, eh);
#pragma unroll
                        for (int jj = 0; jj < vGroup; ++jj) em |= mm[jj] <= eh[jj] ? 1u << (j0 + jj) : 0u;
                    } else {
#pragma unroll
                        for (int jj = 0; jj < vGroup; ++jj) {
                            const int j = j0 + jj;
                            if (j < nvis && range_empty(mm[jj], s_runs + j * kMaxRuns, s_ch[j].nruns)) em |= 1u << j;
                        }
                    }
                    if (homog) {
#pragma unroll
                        for (int jj = 0; jj < vGroup; ++jj) {
                            const int j = j0 + jj;
                            if (j < nvis && (mm[jj] & 0xFFFFu) == (mm[jj] >> 16)) hm |= 1u << j;
                        }
                    }
                    asm volatile("" ::: "memory");
                }
                em = all_of_ray(em);
                if (homog) hm = all_of_ray(hm);
                em &= vismask;
                hm &= ~em;
                if (dl == dend) emask = em;
                const bool all_empty = em == vismask;
                const bool rskip = homog && hm && (em | hm) == vismask;
                // (without skipping, empty nodes are stepped through;
                // render-and-skip changes the image, so it stays on)
                if ((all_empty && !noskip) || rskip) {
                    skip = true;
                    end_nsh = nd.nsh;
                    lcd = dl;
                    rs_node = node;
                    if (!all_empty) rs_mask = hm;
                    break;
                }
            }
            cur_leaf = skip ? kInvalid : leaf;
            lcd = skip ? lcd : D;
#pragma unroll
            for (int a = 0; a < 3; ++a) lc[a] = (iu[a] >> field(end_nsh, a)) << field(end_nsh, a);
        }
        // First sample after k that may lie outside the node (or the volume):
        // the last one inside is found from the exit distance and confirmed
        // by the sampling path's own position test; positions grow
        // monotonically, so those in between are inside too.
        double end;
        {
            double te = INFINITY;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (dd[a] == 0.0) continue;
                const int sh = (int)field(end_nsh, a);
                const int lo_a = (iu[a] >> sh) << sh;
                const int bound = dd[a] > 0.0 ? min(lo_a + (1 << sh), A.dims[a]) : lo_a;
                te = fmin(te, ((double)bound - oo[a]) * lds.inverse(a));
            }
            double kb = fmin(floor(te * A.inv_step), kend);
            auto in_node = [&]() {
                bool in = true;
                const double tk = kb * step;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double ua = fma(tk, dd[a], oo[a]);
                    in = in && ua >= 0.0 && ua < (double)A.dims[a] && ((((int)ua) ^ iu[a]) >> field(end_nsh, a)) == 0;
                }
                return in;
            };
            end = k + 1.0;
            for (int i = 0; i < 2 && kb > k; ++i) {
                if (in_node()) {
                    end = kb + 1.0;
                    break;
                }
                kb -= 1.0;
            }
        }
        if (skip) {
            if constexpr (HOMOG) {
                if (rs_mask) {
                    // The constant mix of the homogeneous channels (in
                    // visible-channel order, as sampled values mix) for the
                    // taken samples k, k + r, .. of the span: up to the
                    // node's exit, the volume's exit (the node may reach
                    // beyond the volume, whose samples are void) and, with
                    // the adaptive step, the next level threshold (r may
                    // change there).  One transparency factor per sample,
                    // so early termination falls on the same sample as
                    // sample by sample; the colour is summed in closed form.
                    float hp = 1.0f, hsa = 0.0f, hsr = 0.0f, hsg = 0.0f, hsb = 0.0f;
                    const uint32_t *rm = gmem(A.meta) + (size_t)rs_node * m;
                    for (int j = 0; j < nvis; ++j) {
                        if (!((rs_mask >> j) & 1u)) continue;
                        const float v = (float)(rm[s_ch[j].c] & 0xFFFFu);
                        float f, al, r, gg, bb;
                        const int e = j * kTfStride + tf_entry(v, s_par->w0[j], s_par->iw[j], f);
                        if (onecol) {
                            al = fmaf(s_tfa[e].y, f, s_tfa[e].x);
                            r = s_par->r[j];
                            gg = s_par->g[j];
                            bb = s_par->b[j];
                        } else {
                            const float4 ta = s_tf[e], tb = s_tf[e + 1];
                            al = fmaf(tb.w - ta.w, f, ta.w);
                            r = fmaf(tb.x - ta.x, f, ta.x);
                            gg = fmaf(tb.y - ta.y, f, ta.y);
                            bb = fmaf(tb.z - ta.z, f, ta.z);
                        }
                        hp *= 1.0f - al;
                        hsa += al;
                        hsr = fmaf(al, r, hsr);
                        hsg = fmaf(al, gg, hsg);
                        hsb = fmaf(al, bb, hsb);
                    }
                    if (adaptive) end = fmin(end, klod);
                    const double rr = ldexp(1.0, rsh);
                    const double n = fmax(ceil((end - k) / rr), 1.0);
                    uint32_t i = 0;
                    end = k + n * rr;
                    if (hsa > 0.0f) {
                        double tau = (double)hp;
                        for (int q = 0; q < rsh; ++q) tau *= tau;
                        const double t0 = Tr;
                        while ((double)i < n && !done) {
                            Tr *= tau;
                            ++i;
                            done = Tr <= one_minus_term;
                        }
                        const double sc = (t0 - Tr) / (double)hsa;
                        Cr = fma(sc, (double)hsr, Cr);
                        Cg = fma(sc, (double)hsg, Cg);
                        Cb = fma(sc, (double)hsb, Cb);
                    } else {
                        i = (uint32_t)n;  // nothing to composite
                    }
                    if (q == 0) {
                        st_samples += i;
                        st_hom += i;
                        st_iters += i;
                    }
                }
            }
            k = end;
            kseg = k;
            return;
        }
        if (!same) {
            cur_lod = lod;
            if (q == 0) ++st_visits;
            missmask = 0;
            if (rates) {
                // the rate of each channel's clamped desired level (fixed within a visit)
                rpk = 0;
                for (int j = 0; j < nvis; ++j) {
                    const ChanLds ch = s_ch[j];
                    rpk |= (uint64_t)field(s_lv[min(max(lod, ch.lo), ch.hi)].raw, 0) << (4 * j);
                }
            }
            // Residency masks of the leaf give each channel the level it
            // samples (finest resident at or above the desired one).
            const uint16_t *lm = gmem(A.mask) + (size_t)leaf * m;
            uint32_t look = vismask & ~emask;  // channels with a resident brick to look up
            bool uniform = false;              // they sample one level, lu0
            int lu0 = 0;
            if (kOwn > 1 && A.ident && A.uni) {
                // one desired level for every channel: AND the masks of all
                // channels (two per word) and test its bit
                lu0 = min(max(lod, A.lo[0]), A.hi[0]);
                uint32_t miss = 0;
#pragma unroll
                for (int g = 0; g < kOwn; g += vGroup) {
                    if (P == 1 && g >= nvis) break;
                    uint32_t v[vGroup / 2 > 0 ? vGroup / 2 : 1];
                    group_read<(vGroup / 2 > 0 ? vGroup / 2 : 1)>((const uint32_t *)(lm + min(own + g, nvis - vGroup)), v);
#pragma unroll
                    for (int i = 0; i < vGroup / 2; ++i) miss |= ~v[i];
                }
                miss = all_of_ray(miss | miss >> 16);
                uniform = !((miss >> lu0) & 1u);
            }
            if (!uniform) {
                const uint32_t want = look;
                uint32_t levels = 0;  // levels sampled, one bit each
                look = 0;
                uint32_t lv0 = 0, lv1 = 0;  // their levels, 4 bits each
#pragma unroll
                for (int g = 0; g < kOwn; g += vGroup) {
                    const int j0 = own + g;
                    if (P == 1 && g >= nvis) break;
                    uint32_t mk[vGroup];
                    if (vGroup > 1 && A.ident) {
                        uint32_t v[vGroup / 2 > 0 ? vGroup / 2 : 1];
                        group_read<(vGroup / 2 > 0 ? vGroup / 2 : 1)>((const uint32_t *)(lm + min(j0, nvis - vGroup)), v);
#pragma unroll
                        for (int jj = 0; jj < vGroup; ++jj) mk[jj] = jj & 1 ? v[jj / 2] >> 16 : v[jj / 2] & 0xFFFFu;
                    } else {
#pragma unroll
                        for (int jj = 0; jj < vGroup; ++jj) mk[jj] = (uint32_t)lm[s_ch[j0 + jj].c];
                    }
#pragma unroll
                    for (int jj = 0; jj < vGroup; ++jj) {
                        const int j = j0 + jj;
                        if ((want >> j) & 1u) {
                            const ChanLds ch = s_ch[j];
                            const int ls = min(max(lod, ch.lo), ch.hi);
                            const uint32_t mj = mk[jj] >> ls;
                            if (!(mj & 1u)) missmask |= 1u << j;
                            if (mj) {
                                const int lu = ls + __builtin_ctz(mj);
                                if (j < 8) lv0 |= (uint32_t)lu << (4 * j);
                                else lv1 |= (uint32_t)lu << (4 * j - 32);
                                look |= 1u << j;
                                levels |= 1u << lu;
                            }
                        }
                    }
                }
                look = all_of_ray(look);
                levels = all_of_ray(levels);
                missmask = all_of_ray(missmask);
                lvpack = (uint64_t)all_of_ray(lv0) | (uint64_t)(NV > 8 ? all_of_ray(lv1) : 0u) << 32;
                uniform = (levels & (levels - 1u)) == 0;
                lu0 = __builtin_ctz(levels | 0x10000u) & 15;
            }
            // Misses are counted by the visits that share the missing
            // channels and the desired bricks: the finest desired brick and
            // the level fix the others.
            if (missmask | pmask) {
                const LevLds lf = s_lv[min(max(lod, A.step_lo), A.step_hi)];
                const uint32_t key = (uint32_t)(iu[0] >> field(lf.sh, 0)) | (uint32_t)(iu[1] >> field(lf.sh, 1)) << 8 |
                                     (uint32_t)(iu[2] >> field(lf.sh, 2)) << 16 | (uint32_t)lod << 24;
                if (missmask != pmask || key != pkey) {
                    // the wave adds them after the visits
                    fpend = npend;
                    fmask = pmask;
                    fkey = pkey;
                    npend = 0;
                    pmask = rates ? 0 : missmask;
                    pkey = key;
                }
            }
            // When every looked-up channel samples one level, its bricks are
            // the same grid cell in each channel: if that cell and level are
            // those of the previous visit, the slots found then still hold
            // (the page table does not change during a frame).
            uint32_t key = kInvalid, cell = 0;
            if (look && uniform) {
                const LevLds lv = s_lv[lu0];
                cell = brick_dense(lv, 0u, 0u, iu[0] >> field(lv.sh, 0), iu[1] >> field(lv.sh, 1),
                                   iu[2] >> field(lv.sh, 2));
                key = cell | ((uint32_t)lu0 << 28);
            }
            const uint32_t reuse = (key != kInvalid && key == last_key) ? have : 0u;
            const uint32_t find = look & ~reuse;
            uint32_t nhave = reuse & look;
            // channels whose slot changes: looked up anew, or no longer sampled
            if (find) {
                uint32_t got = 0, restamp = 0;
#pragma unroll
                for (int g = 0; g < kOwn; g += vGroup) {
                    const int j0 = own + g;
                    if (P == 1 && g >= nvis) break;
                    uint32_t ns[vGroup], cb[vGroup];
                    group_read<vGroup>(s_par->cbase + j0, cb);
#pragma unroll
                    for (int jj = 0; jj < vGroup; ++jj) {
                        const int j = j0 + jj;
                        ns[jj] = kInvalid;
                        if ((find >> j) & 1u) {
                            uint32_t b = cell;
                            if (key == kInvalid) {
                                const LevLds lv = s_lv[(int)((lvpack >> (4 * j)) & 15u)];
                                b = brick_dense(lv, 0u, 0u, iu[0] >> field(lv.sh, 0), iu[1] >> field(lv.sh, 1),
                                                iu[2] >> field(lv.sh, 2));
                            }
                            ns[jj] = gmem(A.pt)[cb[jj] + b];
                        }
                    }
#pragma unroll
                    for (int jj = 0; jj < vGroup; ++jj) {
                        const int j = j0 + jj;
                        if (ns[jj] != kInvalid) {
                            got |= 1u << j;
                            if (!((have >> j) & 1u) || ns[jj] != lds.slot(j)) {
                                // with rates the stamp waits for a sample the channel takes part in
                                if (rates) restamp |= 1u << j;
                                else gmem(A.stamp)[ns[jj]] = A.frame;
                                lds.slot(j) = ns[jj];
                            }
                        }
                    }
                    asm volatile("" ::: "memory");
                }
                nhave |= all_of_ray(got);
                if (rates) stamped &= ~all_of_ray(restamp);
            }
            // a channel without a slot reads slot 0 in the gathers
            for (uint32_t gone = have & ~nhave; gone; gone &= gone - 1u) lds.slot(__builtin_ctz(gone)) = 0;
            have = nhave;
            last_key = key;
            // the ray in the voxels of the segment's level
            uint32_t nsh = 0;
            if (key != kInvalid) {
                const LevLds lv = s_lv[lu0];
                nsh = lv.raw;
                const uint32_t bx = (uint32_t)(iu[0] >> field(lv.sh, 0)) << A.Blog,
                               by = (uint32_t)(iu[1] >> field(lv.sh, 1)) << A.Blog,
                               bz = (uint32_t)(iu[2] >> field(lv.sh, 2)) << A.Blog;
                cbias = (bz * E + by) * E + bx;
            }
            vsh = nsh;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                o[a] = ldexp(oo[a], -(int)field(nsh, a));
                d[a] = ldexp(dd[a], -(int)field(nsh, a));
            }
        }
        // the segment: samples of this leaf at this level
        kseg = fmin(end, klod);
        if (have == 0 && !per_sample) {
            // no channel has a slot here: the segment's samples are counted, not taken
            const double rr = ldexp(1.0, rsh);
            const double n = fmax(ceil(ldexp(kseg - k, -rsh)), 1.0);
            const uint32_t c = (uint32_t)n;
            npend += c;
            if (q == 0) {
                st_samples += c;
                st_nonempty += c * __popc(vismask & ~emask);
                st_iters += c;
            }
            k += n * rr;
            kseg = k;
        }
    };

    // The segment's next P samples: lane q takes the q-th of them, and each
    // lane composites all of them in order.
    auto sample = [&]() {
        const double rr = (double)(1 << rsh);
        const double kq = P == 1 ? k : k + (double)q * rr;
        const bool mine = P == 1 || kq < kseg;
        float prod = 1.0f, sa = 0.0f, sr = 0.0f, sg = 0.0f, sbl = 0.0f;
        // channels taking part in this sample (all of them without rates)
        uint32_t part = vismask;
        if (rates) {
            part = 0;
            const uint32_t kl = (uint32_t)(uint64_t)kq;  // rates are at most 2^15
            for (int j = 0; j < nvis; ++j) {
                const int rs = (int)((rpk >> (4 * j)) & 15u);
                if (!(kl & ((1u << rs) - 1u))) part |= 1u << j;
            }
        }
        if (AOV && A.reqb) {
            // Bricks required per pixel: the desired brick of each channel not
            // empty here that takes part in the sample (a leaf lies in one
            // brick per level).  Along a ray the desired level never decreases
            // and a brick's samples are one interval, so each required brick is
            // one run of equal keys: count the changes.
            uint32_t *rb = A.reqb + ((size_t)py * A.W + px) * (1 + nvis);
            for (int j = 0; j < nvis; ++j) {
                if (((emask >> j) & 1u) || !((part >> j) & 1u)) continue;
                const ChanLds ch = s_ch[j];
                const LevLds lv = s_lv[min(max(lod, ch.lo), ch.hi)];
                const uint32_t key = brick_dense(lv, 0u, 0u, lc[0] >> field(lv.sh, 0), lc[1] >> field(lv.sh, 1),
                                                 lc[2] >> field(lv.sh, 2));
                if (rb[1 + j] != key) {
                    rb[1 + j] = key;
                    rb[0] += 1;
                }
            }
        }
        const uint32_t use = have & part;  // the channels gathered below
        // ---- sample every visible channel
        // Channels are gathered in groups of kGroup: the group's loads are all
        // issued before any of them is used, and two horizontally adjacent
        // voxels come in one load.
        const double t = kq * step;
        uint32_t idx = 0;
        float fr0 = 0.0f, fr1 = 0.0f, fr2 = 0.0f;
        int lprev = -1;
        // in-brick voxel index and fractions where channels sample different levels
        auto in_brick = [&](int lu) {
            const LevLds lv = s_lv[lu];
            uint32_t i0[3];
            float fr[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double u = ldexp(fma(t, d[a], o[a]), -(int)field(lv.raw, a)) + 0.5;
                i0[a] = (uint32_t)((int)u - ((lc[a] >> field(lv.sh, a)) << A.Blog));
                fr[a] = (float)__builtin_amdgcn_fract(u);
            }
            idx = (i0[2] * E + i0[1]) * E + i0[0];
            fr0 = fr[0];
            fr1 = fr[1];
            fr2 = fr[2];
            lprev = lu;
        };
        // Gather, interpolate, classify and mix every channel with a slot.
        // With UNI every such channel reads the visit's one level, whose
        // coordinates are computed before the loop.
        auto sample_channels = [&](auto uni_c) {
            constexpr bool UNI = decltype(uni_c)::value;
#pragma unroll
            for (int g = 0; g < NV; g += kGroup) {
                if (g >= nvis) break;
                uint32_t sw[kGroup], w[kGroup][4];
                float fq[kGroup][3];
                lds.group(g, sw);
                float w0[kGroup], iw[kGroup];
                group_read<kGroup>(s_par->w0 + g, w0);
                group_read<kGroup>(s_par->iw + g, iw);
#pragma unroll
                for (int jj = 0; jj < kGroup; ++jj) {
                    const int j = g + jj;
                    if constexpr (!UNI) {
                        const int lu = (int)((lvpack >> (4 * j)) & 15u);
                        if (((use >> j) & 1u) && lu != lprev) in_brick(lu);
                    }
                    fq[jj][0] = fr0;
                    fq[jj][1] = fr1;
                    fq[jj][2] = fr2;
                    // a channel without a slot reads slot 0 (always inside the
                    // pool) and looks up the zero entry
                    const uint8_t *base = pool + ((uint64_t)sw[jj] * stride + (uint64_t)(idx * (uint32_t)BPV));
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[jj][i] = vpair<BPV>(base + (size_t)((i & 1) * E + (i >> 1) * E * E) * BPV);
                }
                // interpolated value of the group's channel jj
                auto value = [&](int jj) {
                    const float f0 = fq[jj][0], f1 = fq[jj][1], f2 = fq[jj][2];
                    float c[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float v[2];
                        unpack<BPV>(w[jj][i], v);
                        c[i] = fmaf(v[1] - v[0], f0, v[0]);
                    }
                    const float e0 = fmaf(c[1] - c[0], f1, c[0]);
                    const float e1 = fmaf(c[3] - c[2], f1, c[2]);
                    return fmaf(e1 - e0, f2, e0);
                };
                // mixes a channel of opacity al and colour (r, gg, bb); an
                // opacity of zero changes nothing
                auto mix = [&](int j, float al, float r, float gg, float bb) {
                    if (rates) {
                        // the channel stands for r_c base steps: transparency
                        // (1 - alpha)^r_c, colour weight r_c alpha
                        const int rs = (int)((rpk >> (4 * j)) & 15u);
                        float tr = 1.0f - al;
                        for (int q = 0; q < rs; ++q) tr *= tr;
                        const float wt = (float)(1 << rs) * al;
                        prod *= tr;
                        sa += wt;
                        sr = fmaf(wt, r, sr);
                        sg = fmaf(wt, gg, sg);
                        sbl = fmaf(wt, bb, sbl);
                    } else {
                        prod *= 1.0f - al;
                        sa += al;
                        sr = fmaf(al, r, sr);
                        sg = fmaf(al, gg, sg);
                        sbl = fmaf(al, bb, sbl);
                    }
                    if (AOV && A.aov && ((use >> j) & 1u))
                        A.aov[((size_t)py * A.W + px) * L + (UNI ? (int)(last_key >> 28) : (int)((lvpack >> (4 * j)) & 15u))] += 1;
                };
                // table positions of the group, then its table reads, then the mix
                int e[kGroup];
                float f[kGroup];
#pragma unroll
                for (int jj = 0; jj < kGroup; ++jj)
                    e[jj] = (g + jj) * kTfStride + tf_entry(value(jj), w0[jj], iw[jj], f[jj]);
                constexpr uint32_t gm = (1u << kGroup) - 1u;
                if (__any(((use >> g) & gm) != gm)) {
#pragma unroll
                    for (int jj = 0; jj < kGroup; ++jj)
                        if (!((use >> (g + jj)) & 1u)) e[jj] = kTfStride * NV;
                }
                if (onecol) {
                    // Every visible channel has one colour in all its table
                    // entries (the usual stain colouring): its interpolation
                    // returns that colour exactly, so only the opacity is
                    // looked up: one 8-byte read and one multiply-add for two
                    // 16-byte reads and eight operations.
                    float2 ta[kGroup];
                    float r[kGroup], gg[kGroup], bb[kGroup];
#pragma unroll
                    for (int jj = 0; jj < kGroup; ++jj) ta[jj] = s_tfa[e[jj]];
                    group_read<kGroup>(s_par->r + g, r);
                    group_read<kGroup>(s_par->g + g, gg);
                    group_read<kGroup>(s_par->b + g, bb);
#pragma unroll
                    for (int jj = 0; jj < kGroup; ++jj)
                        mix(g + jj, fmaf(ta[jj].y, f[jj], ta[jj].x), r[jj], gg[jj], bb[jj]);
                } else {
#pragma unroll
                    for (int jj = 0; jj < kGroup; ++jj) {
                        const float4 ta = s_tf[e[jj]], tb = s_tf[e[jj] + 1];
                        mix(g + jj, fmaf(tb.w - ta.w, f[jj], ta.w), fmaf(tb.x - ta.x, f[jj], ta.x),
                            fmaf(tb.y - ta.y, f[jj], ta.y), fmaf(tb.z - ta.z, f[jj], ta.z));
                    }
                }
                // the next group's loads are issued after this group is used:
                // bounds the registers held by loads in flight
                asm volatile("" ::: "memory");
            }
        };
        float as = 0.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
        double trr = 1.0, dr = 0.0, dg = 0.0, db = 0.0;  // with opacity correction
        const bool corr = rsh != 0 && !rates;
        if (mine) {
            if (last_key != kInvalid) {
                // one level for every channel with a slot (the visit's lookup key)
                int qi[3];
                float fr[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double u = fma(t, d[a], o[a]) + 0.5;
                    qi[a] = (int)u;
                    fr[a] = (float)__builtin_amdgcn_fract(u);
                }
                idx = ((uint32_t)qi[2] * E + (uint32_t)qi[1]) * E + (uint32_t)qi[0] - cbias;
                fr0 = fr[0];
                fr1 = fr[1];
                fr2 = fr[2];
                sample_channels(std::true_type{});
            } else {
                sample_channels(std::false_type{});
            }
            if (sa > 0.0f) {
                if (!corr) {
                    as = 1.0f - prod;
                    const float sc = as / sa;
                    cr = sr * sc;
                    cg = sg * sc;
                    cb = sbl * sc;
                } else {
                    // opacity correction for a sample standing for r base steps:
                    // transparency prod^r, colour scaled with the opacity
                    trr = (double)prod;
                    for (int i = 0; i < rsh; ++i) trr *= trr;
                    const double sc = (1.0 - trr) / (double)sa;
                    dr = (double)sr * sc;
                    dg = (double)sg * sc;
                    db = (double)sbl * sc;
                }
            }
        }
        uint32_t taken = 0;
        const uint32_t hit = (sa > 0.0f ? 1u : 0u) | (mine ? 2u : 0u);
        auto composite = [&](auto lane_c) {
            constexpr int i = decltype(lane_c)::value;
            const uint32_t h = ray_lane<P, i>(hit);
            if (done || !(h & 2u)) return;
            ++taken;
            if (!(h & 1u)) return;
            if (!corr) {
                Cr = fma(Tr, (double)ray_lane<P, i>(cr), Cr);
                Cg = fma(Tr, (double)ray_lane<P, i>(cg), Cg);
                Cb = fma(Tr, (double)ray_lane<P, i>(cb), Cb);
                Tr *= 1.0 - (double)ray_lane<P, i>(as);
            } else {
                Cr = fma(Tr, ray_lane<P, i>(dr), Cr);
                Cg = fma(Tr, ray_lane<P, i>(dg), Cg);
                Cb = fma(Tr, ray_lane<P, i>(db), Cb);
                Tr *= ray_lane<P, i>(trr);
            }
            done = Tr <= one_minus_term;
        };
        composite(std::integral_constant<int, 0>{});
        if (P == 4) {
            composite(std::integral_constant<int, 1>{});
            composite(std::integral_constant<int, 2>{});
            composite(std::integral_constant<int, 3>{});
        }
        if (!rates) {
            npend += taken;
        } else {
            // misses and stamps per sample (a visit's samples differ in which
            // channels take part); the wave adds the misses after the samples
            const bool counts = P == 1 || (uint32_t)q < taken;
            smiss = counts ? missmask & part : 0u;
            uint32_t sp = counts ? have & part & ~stamped : 0u;
            const uint32_t now = all_of_ray(sp);
            while (sp) {
                const int j = __builtin_ctz(sp);
                sp &= sp - 1u;
                gmem(A.stamp)[lds.slot(j)] = A.frame;
            }
            stamped |= now;
        }
        if (P == 1 || (uint32_t)q < taken) {
            ++st_samples;
            st_nonempty += __popc(vismask & ~emask & part);
            st_reads += __popc(use);
        }
        // the next sample: with the adaptive step the next multiple of r (the
        // level only grows along the ray, so no grid point lies in between)
        k += P == 1 ? rr : rr * (double)taken;
    };

    // Rays of a wave keep together, so that their gathers share cache lines: a
    // ray samples while its index is at most klim, counted from the last ray
    // of the wave (as of when the limit was last set).  The distance is in
    // whole groups of P samples, 1.25 of them per sample that a pixel's
    // footprint spans: where neighbouring rays are far apart their samples
    // share few lines anyway and fewer waits count more (this against always
    // one group: 16 channels 1080p at half a voxel a pixel, where it is one
    // group, 41.0 ms both, and 42.0 with another group; 512 x 512, 4 channels,
    // two voxels a pixel 2.10 against 2.35; 720p, 8 channels, adaptive 3.25
    // against 4.27).
    // Visits wait until kVisitLanes lanes need one or no ray can sample: a
    // visit is a chain of dependent loads and several hundred instructions,
    // whatever the number of lanes that take part (every visit at once, at 8,
    // 16 and 24 lanes: 512 x 512, 4 channels 2.42 ms, 2.33, 2.15, 2.10; 720p,
    // 8 channels, adaptive 3.64, 3.46, 3.31, 3.25; 455 x 256, 16 channels,
    // six voxels a pixel 2.68, 2.62, 2.78, 2.99).
    constexpr int kVisitLanes = 24;
    double klim = -1.0;
    if ((threadIdx.x & 63u) < kMissEntries) lds.miss[3 * (threadIdx.x & 63u) + 1] = 0;
    wave_sync();
    src.init();
    while (true) {
        const bool fin = has && (done || k > kend);
        if (__any(fin)) {
            flush(fin && q == 0 ? npend : 0u, pmask, pkey);
            if (fin) finish();
        }
        if (!__any(has)) {
            int x = 0, y = 0;
            bool v = false;
            if (!src.next(x, y, v)) break;
            start(x, y, v);
            wave_sync();
        }
        const bool active = has && !done && k <= kend;
        const bool wv = active && k >= kseg;
        const uint64_t bv = __ballot(wv);
        bool ws = active && !wv && k <= klim;
        uint64_t bs = __ballot(ws);
        if (!bs) {
            // (the minimum is taken by all lanes of the wave, not under a branch)
            // the limit bounds the lanes' distance only: a rounded index does
            const float kmin = wave_min(active ? (float)k : 3.0e38f);
            const float groups = floorf(1.25f * fmaf(kmin, A.win_k, A.win_0) + 0.5f);
            klim = (double)(kmin + (float)P * fmaxf(groups, 1.0f) - 1.0f);
            ws = active && !wv && (k <= klim || !bv);
            bs = __ballot(ws);
        }
        if (!(bv | bs)) continue;  // rays that just began without a sample
        if (bv && (!bs || __popcll(bv) >= kVisitLanes)) {
            wave_sync();
            if (wv) visit();
            wave_sync();
            flush(q == 0 ? fpend : 0u, fmask, fkey);
            fpend = 0;
            continue;
        }
        ++st_iters;  // a stepping iteration of the wave (lane busy or idle)
        if (ws) sample();
        if (rates) {
            flush(smiss ? 1u : 0u, smiss, pkey);
            smiss = 0;
        }
    }
    // the table's sums
    for (int i = 0; i < kMissEntries; ++i) {
        const uint32_t *e = lds.miss + 3 * i;
        if (e[1]) count_misses(e[0], e[1], e[2]);
    }
    stats[0] = st_samples;
    stats[1] = st_reads;
    stats[2] = st_miss;
    stats[3] = st_visits;
    stats[4] = st_nonempty;
    stats[5] = st_iters;
    stats[6] = st_hom;
}

// Workgroup set-up: stage the frame's transfer functions, zero-alpha runs,
// channel parameters, per-level brick tables and per-level node tables in
// LDS.  A wave looks over a channel's table with four 64-entry ballots (a
// scan by one lane, entry after entry through LDS, was 10 us of a small
// frame).  Where every visible table has one colour, the tables are staged as
// (opacity, step) pairs.  Ends with a workgroup barrier.
template <int NV>
__device__ __forceinline__ void stage_frame(const RenderArgs &A, float4 *s_tf, ChanLds *s_ch, ChanPar<NV> *s_par,
                                            uint32_t *s_runs, LevLds *s_lv, NodeLds *s_nd) {
    const int nvis = A.nvis;
    const unsigned t = threadIdx.x;
    const int lane = (int)(t & 63u), wave = (int)(t >> 6), waves = (int)(blockDim.x >> 6);
    const float4 *tf = gmem(A.tf);
    if (t < (unsigned)A.L) {
        LevLds lv;
        lv.raw = A.lsh[t];
        lv.sh = lv.raw + (uint32_t)A.Blog * 0x010101u;
        lv.loff = A.loff[t];
        lv.nbx = A.nbx[t];
        lv.nbxy = A.nbx[t] * A.nby[t];
        lv.K = A.K[t];
        lv.dd = A.dd[t];
        s_lv[t] = lv;
    }
    if (t < (unsigned)NV && t >= (unsigned)nvis) {
        s_par->w0[t] = s_par->iw[t] = 0.0f;
        s_par->r[t] = s_par->g[t] = s_par->b[t] = 0.0f;
        s_par->ehi[t] = s_par->cbase[t] = 0;
        s_ch[t].c = 0;
    }
    if (t >= 32 && t < 35) {
        const int a = (int)t - 32;
        s_par->ax[a] = {A.eye[a], A.F[a], A.R[a], A.U[a], A.sp[a], (double)A.dims[a]};
    }
    if (t >= 64 && t < 64u + (unsigned)A.depth + 1u) {
        const unsigned dl = t - 64;
        NodeLds nd;
        nd.nsh = A.nsh[dl];
        nd.nlg = A.nlg[dl];
        nd.noff = A.noff[dl];
        s_nd[dl] = nd;
    }
    for (int j = wave; j < nvis; j += waves) {
        const float4 e0 = tf[j * 256];
        uint64_t zero[4], same = ~0ull;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 e = tf[j * 256 + 64 * q + lane];
            zero[q] = __ballot(e.w == 0.0f);
            // (x - x is zero for finite values only)
            same &= __ballot(e.x == e0.x && e.y == e0.y && e.z == e0.z && (e.x - e.x) + (e.y - e.y) + (e.z - e.z) == 0.0f);
        }
        if (lane == 0) {
            ChanLds ch;
            ch.c = A.vis[j];
            ch.lo = A.lo[j];
            ch.hi = A.hi[j];
            s_par->w0[j] = A.w0[j];
            s_par->iw[j] = A.iw[j];
            s_par->r[j] = e0.x;
            s_par->g[j] = e0.y;
            s_par->b[j] = e0.z;
            s_par->cbase[j] = (uint32_t)A.vis[j] * A.per_channel;
            ch.onecol = same == ~0ull;
            ch.nruns = build_runs(zero, A.W0[j], A.W1[j], s_runs + j * kMaxRuns);
            const uint32_t r0 = s_runs[j * kMaxRuns];
            ch.ehi = (ch.nruns == 1 && (r0 & 0xFFFFu) == 0) ? (r0 >> 16) : 0xFFFFFFFFu;
            s_par->ehi[j] = (r0 & 0xFFFF0000u) | 0xFFFFu;
            ch.single = 0;
            s_ch[j] = ch;
        }
    }
    __syncthreads();
    uint32_t all = 1, one = 1;
    for (int j = 0; j < nvis; ++j) {
        all &= s_ch[j].ehi != 0xFFFFFFFFu ? 1u : 0u;
        one &= s_ch[j].onecol;
    }
    if (t < 2) {
        if (one) ((float2 *)s_tf)[NV * kTfStride + t] = make_float2(0.0f, 0.0f);
        else s_tf[NV * kTfStride + t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    if (one) {
        float2 *tfa = (float2 *)s_tf;
        for (int i = (int)t; i < nvis * kTfStride; i += (int)blockDim.x) {
            const int c = i / kTfStride, e = min(i - c * kTfStride, 255);
            const float a = tf[c * 256 + e].w;
            tfa[i] = make_float2(a, tf[c * 256 + min(e + 1, 255)].w - a);
        }
    } else {
        for (int i = (int)t; i < nvis * kTfStride; i += (int)blockDim.x) {
            const int c = i / kTfStride, e = min(i - c * kTfStride, 255);
            s_tf[i] = tf[c * 256 + e];
        }
    }
    __syncthreads();
    if (t < (unsigned)nvis) {
        s_ch[t].single = all;
        s_ch[t].onecol = one;
    }
    __syncthreads();
}

}  // namespace ro
