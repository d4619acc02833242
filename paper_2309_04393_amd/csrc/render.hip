// Ray-guided mixed-resolution multi-channel ray casting over the residency
// octree (Sec. 6.1, Alg. 1; Sec. 6.2; Sec. 7 implementation notes).
//
// Four lanes per ray; persistent 768-lane workgroups (one per CU) whose waves
// take units of 4 x 4 pixels from per-XCD queues.  A ray alternates between
// visits of a leaf (its four lanes share the leaf's channels) and samples
// (each lane takes one of the ray's next four).
// Sample positions and every integer decision derived from them (box, leaf,
// brick, level) are computed in FP64; interpolation, transfer functions and
// the channel mix in FP32; the compositing state in FP64, sample after
// sample, so the image does not depend on the number of lanes (one per ray,
// the diagnostic outputs, and four gave the same bits in 28 frames compared).
// Per ray, the state of the current (leaf, level) visit is cached: which
// channels are empty there, the slot each channel samples, and which channels
// miss their desired brick; misses are summed while the missing channels and
// their desired bricks stay the same, over the rays of a wave, before they
// reach the device counters.
//
// Every table a lane indexes with a lane-dependent value (channel
// parameters, zero-alpha runs, per-level brick grid and LOD thresholds,
// per-level node grid, transfer functions) is staged in LDS at workgroup
// start; kernel arguments are only read with uniform indices.
#include <math.h>
#include <string.h>

#include "render_core.h"

namespace ro {

// Workgroups of kRenderLanes lanes (768: 3 waves per SIMD, up to 168 VGPRs),
// one per CU: one copy of the frame's LDS tables plus the per-ray words.
// 1024 lanes (4 waves per SIMD, 128 VGPRs) spill and measured 45 % slower on
// the 16-channel 1080p frame and twice as slow on 512 x 512 with 4 channels,
// 512 lanes 5 % slower on both (with one lane per ray).
//
// What bounds the frame kernel: on the 16-channel 1080p frame (1024 x 1024 x
// 192 voxels, half a voxel per pixel, 8.4e8 ray samples) 41.0 ms against 58
// with one lane per ray in lockstep.  Vector instructions fill two thirds of
// the issue slots and the address and tag units are busy throughout: 1.2e9
// gathers of 64 lanes, each 18.5 tag lookups.  Gathers of single 16-bit
// voxels (8 per channel instead of 4) touch as many lines each and took
// 70 ms; aligned addresses alone (wrong voxels) save 2 %.  Frames of a few
// thousand units are bound by their longest rays: four lanes per ray cut
// those (512 x 512, 4 channels: 5.0 ms -> 2.1; 24 x 24, 16 channels: 8.2 ->
// 1.16, and 0.73 with its units in parts, see render_device; 64 x 64, one
// channel: 0.58 -> 0.13).  Rays that end at once are bound by vector
// instructions: a unit of 16 of them is 1300 to 1900, 400 of them its set-up.
// A full-HD frame of rays that all end within eight samples is what one lane
// per ray was better at (4 channels, 2.4 samples a pixel 0.34 ms, 0.36 now; 1
// channel, 7.6 samples 0.45 and 0.53; 16 channels, 0.6 samples 0.35 and 0.43).
//
// Scratch: none with up to eight channels but for 8 bytes a lane in one
// instance; with 16 channels 28 to 32, three addresses that are read where
// sums of misses leave for the counters, not in the channel loop.  Render-and-
// skip keeps 28 to 60, per-channel rates 16 to 56 (none with one channel), the
// diagnostic kernel 24 to 60.

// Persistent grid (one workgroup per CU) whose waves take units of pixels
// from a device counter independently of each other, so a CU never waits
// for the slowest wave of a workgroup before taking new work.
template <int NV, int BPV, bool AOV, int EC, int EXT, int P>
__global__ void __launch_bounds__(kRenderLanes) __attribute__((amdgpu_waves_per_eu(kRenderLanes / 256)))
    k_render(const RenderArgs A, uint32_t *counter, uint32_t n_blocks, uint32_t tiles_x, uint32_t chunk,
             uint32_t n_waves, uint32_t split, uint32_t take) {
    extern __shared__ float4 s_tf[];  // tables, per-ray words, miss tables (render_lds_bytes)
    __shared__ ChanLds s_ch[NV];
    __shared__ ChanPar<NV> s_par;
    __shared__ uint32_t s_runs[NV * kMaxRuns];
    __shared__ LevLds s_lv[kMaxL];
    __shared__ NodeLds s_nd[kMaxD + 1];
    __shared__ UnitLds s_wg;

    if (threadIdx.x == 0) s_wg.clear();
    stage_frame<NV>(A, s_tf, s_ch, &s_par, s_runs, s_lv, s_nd);
    if ((threadIdx.x >> 6) >= n_waves) return;  // a small frame: its blocks are spread over the CUs

    UnitQueue<P> q;
    q.counter = counter;
    q.n_units = (n_blocks * P) << split;
    q.offset = 0;
    q.tiles_x = tiles_x;
    q.n_queues = RO_QUEUES;
    q.chunk = chunk;
    q.split = P == 4 ? split : 0;
    q.take = take;
    q.wg = &s_wg;
    q.W = A.W;
    q.H = A.H;
    uint32_t st[7] = {0, 0, 0, 0, 0, 0, 0};
    render_rays<NV, BPV, AOV, EC, EXT, P>(A, q, s_tf, s_ch, &s_par, s_runs, s_lv, s_nd, st);
    if (A.stats) {
        // whole waves are here: reduce over the wave, one atomic per wave
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            uint32_t v = st[j];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if ((threadIdx.x & 63) == 0 && v) atomicAdd(&A.stats[j], (unsigned long long)v);
        }
    }
}

// Lanes per ray: four, each taking the next of four consecutive samples of
// its ray and a quarter of a visit's channels; the diagnostic outputs are
// recorded sample after sample and take one lane per ray.
constexpr int lanes_per_ray(bool aov) { return aov ? 1 : 4; }

struct QueueLaunch {
    dim3 grid;
    uint32_t *counter;
    uint32_t n_blocks, tiles_x, chunk, n_waves, split, take;
};

template <int NV, int BPV, bool AOV, int EC, int EXT>
static hipError_t launch_one(const RenderArgs &A, const QueueLaunch &Q, hipStream_t s) {
    constexpr int P = lanes_per_ray(AOV);
    const size_t lds = render_lds_bytes(NV, P);
    hipError_t e = hipFuncSetAttribute((const void *)k_render<NV, BPV, AOV, EC, EXT, P>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_render<NV, BPV, AOV, EC, EXT, P>), Q.grid, dim3(kRenderLanes), lds, s, A, Q.counter, Q.n_blocks,
                       Q.tiles_x, Q.chunk, Q.n_waves, Q.split, Q.take);
    return hipGetLastError();
}

// Compile-time brick edges: 32^3 and 16^3 bricks with their halo (the AOV
// diagnostic output takes the generic kernel).
// Render-and-skip of homogeneous nodes (EXT bit 0) and per-channel sampling
// rates (EXT bit 1) have instantiations of their own, so the kernels that do
// not take them carry none of their code.
template <int NV, int BPV, int EXT>
static hipError_t launch_edge(const RenderArgs &A, const QueueLaunch &Q, hipStream_t s) {
    if (A.E == 34) return launch_one<NV, BPV, false, 34, EXT>(A, Q, s);
    if (A.E == 18) return launch_one<NV, BPV, false, 18, EXT>(A, Q, s);
    return launch_one<NV, BPV, false, 0, EXT>(A, Q, s);
}

// The instantiations are compiled in five parts, one object file each
// (RO_PART 0 to 4; unset: all in one): the host side, 8- and 16-bit voxels without
// and with the options.
template <int BPV>
hipError_t launch_plain(const RenderArgs &A, const QueueLaunch &Q, hipStream_t s);
template <int BPV>
hipError_t launch_options(const RenderArgs &A, bool aov, const QueueLaunch &Q, hipStream_t s);

#if !defined(RO_PART) || RO_PART == 1 || RO_PART == 2
template <int BPV>
hipError_t launch_plain(const RenderArgs &A, const QueueLaunch &Q, hipStream_t s) {
    if (A.nvis <= 1) return launch_edge<1, BPV, 0>(A, Q, s);
    if (A.nvis <= 2) return launch_edge<2, BPV, 0>(A, Q, s);
    if (A.nvis <= 4) return launch_edge<4, BPV, 0>(A, Q, s);
    if (A.nvis <= 8) return launch_edge<8, BPV, 0>(A, Q, s);
    return launch_edge<16, BPV, 0>(A, Q, s);
}
#if !defined(RO_PART) || RO_PART == 1
template hipError_t launch_plain<1>(const RenderArgs &, const QueueLaunch &, hipStream_t);
#endif
#if !defined(RO_PART) || RO_PART == 2
template hipError_t launch_plain<2>(const RenderArgs &, const QueueLaunch &, hipStream_t);
#endif
#endif

#if !defined(RO_PART) || RO_PART == 3 || RO_PART == 4
template <int NV, int BPV>
static hipError_t launch_opt(const RenderArgs &A, bool aov, const QueueLaunch &Q, hipStream_t s) {
    if (aov) return launch_one<NV, BPV, true, 0, 3>(A, Q, s);
    if (A.flags & RO_RENDER_HOMOGENEOUS) return launch_edge<NV, BPV, 1>(A, Q, s);
    return launch_edge<NV, BPV, 2>(A, Q, s);
}

template <int BPV>
hipError_t launch_options(const RenderArgs &A, bool aov, const QueueLaunch &Q, hipStream_t s) {
    if (A.nvis <= 1) return launch_opt<1, BPV>(A, aov, Q, s);
    if (A.nvis <= 2) return launch_opt<2, BPV>(A, aov, Q, s);
    if (A.nvis <= 4) return launch_opt<4, BPV>(A, aov, Q, s);
    if (A.nvis <= 8) return launch_opt<8, BPV>(A, aov, Q, s);
    return launch_opt<16, BPV>(A, aov, Q, s);
}
#if !defined(RO_PART) || RO_PART == 3
template hipError_t launch_options<1>(const RenderArgs &, bool, const QueueLaunch &, hipStream_t);
#endif
#if !defined(RO_PART) || RO_PART == 4
template hipError_t launch_options<2>(const RenderArgs &, bool, const QueueLaunch &, hipStream_t);
#endif
#endif

#if !defined(RO_PART) || RO_PART == 0
template <int BPV>
static hipError_t launch_bpv(const RenderArgs &A, bool aov, const QueueLaunch &Q, hipStream_t s) {
    if (aov || (A.flags & (RO_RENDER_HOMOGENEOUS | RO_RENDER_CHANNEL_RATES)))
        return launch_options<BPV>(A, aov, Q, s);
    return launch_plain<BPV>(A, Q, s);
}

// Kernel arguments of one frame (validated by the caller).
ro_status build_render_args(ro_octree *tr, const ro_frame_desc *fd, float *rgba, RenderArgs &A) {
    const ro_cache *c = tr->cache;
    const VolGeo &g = c->vol->g;
    const TreeGeo &T = tr->t;
    memset(&A, 0, sizeof(A));
    for (int k = 0; k < 3; ++k) {
        A.dims[k] = g.dims[k];
        A.sp[k] = g.spacing[k];
        A.eye[k] = fd->eye[k];
        A.F[k] = fd->forward[k];
        A.R[k] = fd->right[k];
        A.U[k] = fd->up[k];
    }
    A.m = g.m;
    A.L = g.L;
    A.Blog = g.Blog;
    A.E = g.E;
    A.depth = T.depth;
    A.start_level = fd->start_level >= 0 ? fd->start_level : tr->desc.start_level;
    A.per_channel = g.per_channel;
    A.slot_stride = g.slot_stride;
    A.tx = fd->tx;
    A.ty = fd->ty;
    A.step = fd->step;
    A.inv_step = 1.0 / fd->step;
    A.proj = fd->projection;
    A.W = fd->width;
    A.H = fd->height;
    for (int l = 0; l < g.L; ++l) {
        A.lsh[l] = (uint32_t)g.lshift[l][0] | ((uint32_t)g.lshift[l][1] << 8) | ((uint32_t)g.lshift[l][2] << 16);
        A.loff[l] = g.loff[l];
        A.nbx[l] = (uint32_t)g.nb[l][0];
        A.nby[l] = (uint32_t)g.nb[l][1];
    }
    for (int d = 0; d <= T.depth; ++d) {
        A.nsh[d] = (uint32_t)T.nshift[d][0] | ((uint32_t)T.nshift[d][1] << 8) | ((uint32_t)T.nshift[d][2] << 16);
        A.nlg[d] = (uint32_t)T.nlog[d][0] | ((uint32_t)T.nlog[d][1] << 8) | ((uint32_t)T.nlog[d][2] << 16);
        A.noff[d] = T.noff[d];
    }
    // desired level thresholds: level l from the first sample k with
    // k * step >= D_l, D_l = s_l / (lod_bias * 2 ty / H)
    const double pix = 2.0 * fd->ty / fd->height;
    for (int l = 0; l < kMaxL; ++l) A.K[l] = kInvalid;
    A.K[0] = 0;
    for (int l = 1; l < g.L; ++l) {
        const double s_l = (double)(1 << g.lshift[l][0]) * g.spacing[0];
        if (fd->projection == RO_PROJ_ORTHO) {
            A.K[l] = fd->lod_bias * pix >= s_l ? 0u : kInvalid;
        } else {
            const double Dl = s_l / (fd->lod_bias * pix);
            const double q = ceil(Dl / fd->step);
            if (!(q < 4.0e9)) {
                A.K[l] = kInvalid;
                continue;
            }
            long long kk = (long long)q;
            while (kk > 0 && (double)(kk - 1) * fd->step >= Dl) --kk;
            while ((double)kk * fd->step < Dl) ++kk;
            A.K[l] = kk < 0xFFFFFFFFll ? (uint32_t)kk : kInvalid;
        }
    }
    // traversal depth from the step (Alg. 1 chooseTraversalDepth): for the
    // step of level l, the deepest node whose smallest world extent is at
    // least the distance between samples, f_l * step
    for (int l = 0; l < kMaxL; ++l) A.dd[l] = (uint32_t)T.depth;
    if ((fd->flags & RO_RENDER_TRAVERSAL_DEPTH) && (fd->flags & RO_RENDER_ADAPTIVE_STEP)) {
        for (int l = 0; l < g.L; ++l) {
            const double dist = (double)(1 << g.lshift[l][0]) * fd->step;
            int d = T.depth;
            while (d > 0) {
                double ext = INFINITY;
                for (int a = 0; a < 3; ++a) ext = fmin(ext, (double)(1ll << T.nshift[d][a]) * g.spacing[a]);
                if (ext >= dist) break;
                --d;
            }
            A.dd[l] = (uint32_t)d;
        }
    }
    A.nvis = fd->n_vis;
    A.ident = fd->n_vis == g.m && g.m % 4 == 0;
    for (int j = 0; j < fd->n_vis; ++j) A.ident = A.ident && fd->vis[j] == j;
    A.uni = 1;
    for (int j = 0; j < fd->n_vis; ++j) A.uni = A.uni && fd->lod_lo[j] == fd->lod_lo[0] && fd->lod_hi[j] == fd->lod_hi[0];
    // min_c clamp(l, lo_c, hi_c) = clamp(l, min_c lo_c, min_c hi_c)
    A.step_lo = A.step_hi = kMaxL;
    for (int j = 0; j < fd->n_vis; ++j) {
        A.step_lo = fd->lod_lo[j] < A.step_lo ? fd->lod_lo[j] : A.step_lo;
        A.step_hi = fd->lod_hi[j] < A.step_hi ? fd->lod_hi[j] : A.step_hi;
    }
    for (int j = 0; j < fd->n_vis; ++j) {
        A.vis[j] = fd->vis[j];
        A.lo[j] = fd->lod_lo[j];
        A.hi[j] = fd->lod_hi[j];
        A.W0[j] = fd->win_lo[j];
        A.W1[j] = fd->win_hi[j];
        A.w0[j] = (float)(fd->win_lo[j] / 256.0);
        A.iw[j] = (float)(256.0 / ((double)fd->win_hi[j] - (double)fd->win_lo[j]));
    }
    A.win_k = fd->projection == RO_PROJ_ORTHO ? 0.0f : (float)pix;
    A.win_0 = fd->projection == RO_PROJ_ORTHO ? (float)(pix / fd->step) : 0.0f;
    A.term = fd->term_alpha;
    A.frame = fd->frame;
    A.flags = fd->flags;
    A.slots = (const uint8_t *)c->b.slots;
    A.pt = c->b.page_table;
    A.cnt = c->b.counters;
    A.stamp = c->b.stamps;
    A.meta = tr->b.node_meta;
    A.mask = tr->b.node_mask;
    A.tf = (const float4 *)fd->tf_dev;
    A.rgba = rgba;
    A.aov = (fd->flags & RO_RENDER_AOV) ? fd->aov_dev : nullptr;
    A.reqb = (fd->flags & RO_RENDER_BRICKS) ? fd->bricks_dev : nullptr;
    A.nodes = (fd->flags & RO_RENDER_NODES) ? fd->nodes_dev : nullptr;
    A.stats = fd->stats_dev;
    return RO_OK;
}

ro_status render_device(ro_octree *tr, const ro_frame_desc *fd, float *rgba, hipStream_t s) {
    const VolGeo &g = tr->cache->vol->g;
    RenderArgs A;
    ro_status st = build_render_args(tr, fd, rgba, A);
    if (st) return st;
    int dev = 0, ncu = 0;
    RO_HIP(hipGetDevice(&dev));
    RO_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    QueueLaunch Q;
    const uint32_t tiles_x = (uint32_t)(fd->width + 31) / 32, tiles_y = (uint32_t)(fd->height + 31) / 32;
    Q.tiles_x = tiles_x;
    Q.n_blocks = tiles_x * tiles_y * 16;
    // the unit counters are at the end of the octree's scratch
    // buffer (the residency update's lists use the rest); cleared by a kernel, not a
    // memset
    Q.counter = (uint32_t *)((uint8_t *)tr->b.scratch + tr->scratch_bytes - kFrameTail);
    Q.grid = dim3((unsigned)(ncu > 0 ? ncu : 256));
    // a frame with fewer units of pixels than the chip has waves uses as many
    // waves of each workgroup as it has units per CU (64 x 64 pixels: 0.135 ms,
    // 0.149 where the waves that come first take them all), and deals its
    // blocks in smaller chunks, whole 32 x 32 tiles of them
    const int p = lanes_per_ray((fd->flags & (RO_RENDER_AOV | RO_RENDER_BRICKS | RO_RENDER_NODES)) != 0);
    const uint32_t n_units = Q.n_blocks * (uint32_t)p;
    Q.split = 0;
    // and where that leaves SIMDs without a wave, a wave takes a part of a
    // unit's pixels: fewer rays in a wave have fewer steps that are not their
    // own (one part against several up to a wave per SIMD, one channel 24 x
    // 24 and 64 x 64: 173 us to 107, 170 to 135; 16 channels 24 x 24: 1.16 ms
    // to 0.73; up to two waves per SIMD took 10 % less for 64 x 64 with 16
    // channels, but 10 % more for 128 x 128)
    if (p == 4)
        while (Q.split < 4 && ((uint64_t)n_units << (Q.split + 1)) <= (uint64_t)Q.grid.x * 4) ++Q.split;
    const uint32_t per_cu = ((n_units << Q.split) + Q.grid.x - 1) / Q.grid.x;
    Q.n_waves = per_cu < kRenderLanes / 64 ? per_cu : kRenderLanes / 64;
    Q.chunk = (queue_chunk(Q.n_blocks) * (uint32_t)p) << Q.split;
    Q.take = p == 4 ? units_at_once(n_units, Q.grid.x * (kRenderLanes / 64)) : 1;
    st = launch_fill_u32(Q.counter, (uint64_t)RO_QUEUES * kQueueStride, 0u, s);
    if (st) return st;
    // the diagnostic outputs (per-level reads, required bricks) take the AOV kernel
    const bool aov = (fd->flags & (RO_RENDER_AOV | RO_RENDER_BRICKS | RO_RENDER_NODES)) != 0;
    RO_HIP(g.bpv == 1 ? launch_bpv<1>(A, aov, Q, s) : launch_bpv<2>(A, aov, Q, s));
    return RO_OK;
}
#endif  // host part

}  // namespace ro
