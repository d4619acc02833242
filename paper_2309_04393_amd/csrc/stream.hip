// Streaming kernels: request compaction, usage readback, LRU slot
// selection, page-table update and brick scatter (Sec. 4: requests copied to
// the CPU under a global limit; Sec. 5.3: slot selection with LRU eviction).
#include <string.h>

#include <algorithm>
#include <mutex>

#include "common.h"

namespace ro {

// ------------------------------------------------------------------- fills

template <typename T>
__global__ void k_fill(T *__restrict__ p, uint64_t n, T v) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

template <typename T>
static ro_status fill(T *p, uint64_t n, T v, hipStream_t s) {
    if (n == 0) return RO_OK;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    RO_HIP(hipGetLastError());
    return RO_OK;
}

ro_status launch_fill_u32(uint32_t *p, uint64_t n, uint32_t v, hipStream_t s) { return fill(p, n, v, s); }
ro_status launch_fill_u16(uint16_t *p, uint64_t n, uint16_t v, hipStream_t s) { return fill(p, n, v, s); }
ro_status launch_fill_u8(uint8_t *p, uint64_t n, uint8_t v, hipStream_t s) { return fill(p, n, v, s); }

// ----------------------------------------------------------- lists to send

ro_status SentList::wait() {
    const int was = state;
    state = kIdle;
    if (was == kMarked) RO_HIP(hipEventSynchronize(used));
    if (was == kSent) RO_HIP(hipStreamSynchronize(stream));
    return RO_OK;
}

ro_status SentList::make(size_t n, hipStream_t s, uint8_t **out) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    RO_HIP(hipStreamIsCapturing(s, &cap));
    RO_CHECK(cap == hipStreamCaptureStatusNone, RO_E_STATE, "the stream is being captured");
    ro_status st = wait();
    if (st) return st;
    if (!used) RO_HIP(hipEventCreateWithFlags(&used, hipEventDisableTiming));
    try {
        buf.resize(n);
    } catch (...) {
        RO_CHECK(false, RO_E_NOMEM, "out of host memory");
    }
    stream = s;
    *out = buf.data();
    return RO_OK;
}

ro_status SentList::send(void *dev) {
    state = kSent;
    RO_HIP(hipMemcpyAsync(dev, buf.data(), buf.size(), hipMemcpyHostToDevice, stream));
    return RO_OK;
}

void SentList::mark() {
    // (without the event the next list waits for the stream)
    if (state == kSent && hipEventRecord(used, stream) == hipSuccess) state = kMarked;
}

// ------------------------------------------------------ block-level helpers

// Exclusive prefix sum over the block (blockDim.x == 256, 4 waves of 64):
// wave-level via ballot-free shuffles, then across waves through LDS.
__device__ inline uint32_t block_excl_scan_256(uint32_t v, uint32_t *lds4, uint32_t *total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds4[wid] = x;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t t = lds4[w];
        if (w < wid) base += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return base + x - v;
}

// ------------------------------------------------------ request compaction

// Four counters of a thread, in one load where the array allows it (a score
// array is the caller's); zero past the end.
__device__ inline uint4 load_four(const uint32_t *__restrict__ arr, uint64_t base, uint64_t n) {
    if (base + 4 <= n && ((uintptr_t)arr & 15) == 0) return *(const uint4 *)(arr + base);
    uint4 v = {0, 0, 0, 0};
    if (base < n) v.x = arr[base];
    if (base + 1 < n) v.y = arr[base + 1];
    if (base + 2 < n) v.z = arr[base + 2];
    if (base + 3 < n) v.w = arr[base + 3];
    return v;
}

// Sum over the block of 256, the same in every thread.
__device__ inline unsigned long long block_sum_256(unsigned long long v, unsigned long long *lds4) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
    __syncthreads();
    v = lds4[0] + lds4[1] + lds4[2] + lds4[3];
    __syncthreads();
    return v;
}

// Result of a compaction, read back in one copy.
struct CompactTotals {
    unsigned long long sum;
    uint32_t n;
    uint32_t pad;
};

// Per block of 1024 counters: number of nonzero counters and the sum of all.
__global__ void __launch_bounds__(256) k_req_count(const uint32_t *__restrict__ cnt, uint64_t n,
                                                   uint32_t *__restrict__ blk,
                                                   unsigned long long *__restrict__ sums) {
    __shared__ unsigned long long lds[4];
    const uint4 v = load_four(cnt, (uint64_t)blockIdx.x * 1024 + threadIdx.x * 4, n);
    const uint32_t nz = (v.x != 0) + (v.y != 0) + (v.z != 0) + (v.w != 0);
    const unsigned long long tot = block_sum_256(nz, lds);
    const unsigned long long sum = block_sum_256((unsigned long long)v.x + v.y + v.z + v.w, lds);
    if (threadIdx.x == 0) {
        blk[blockIdx.x] = (uint32_t)tot;
        sums[blockIdx.x] = sum;
    }
}

// Exclusive scan of nblk block counts by one block; writes offsets and the
// grand total at offs[nblk].  With out, the totals of the counts and of sums.
__global__ void __launch_bounds__(256) k_scan_blocks(const uint32_t *__restrict__ blk, uint32_t nblk,
                                                     uint32_t *__restrict__ offs,
                                                     const unsigned long long *__restrict__ sums,
                                                     CompactTotals *__restrict__ out) {
    __shared__ uint32_t lds[4];
    __shared__ unsigned long long lds8[4];
    uint32_t carry = 0;
    unsigned long long sum = 0;
    for (uint32_t b0 = 0; b0 < nblk; b0 += 256) {
        uint32_t i = b0 + threadIdx.x;
        uint32_t v = i < nblk ? blk[i] : 0;
        if (out && i < nblk) sum += sums[i];
        uint32_t tot;
        uint32_t e = block_excl_scan_256(v, lds, &tot);
        if (i < nblk) offs[i] = carry + e;
        carry += tot;
    }
    if (threadIdx.x == 0) offs[nblk] = carry;
    if (!out) return;
    sum = block_sum_256(sum, lds8);
    if (threadIdx.x == 0) *out = {sum, carry, 0};
}

// Writes the ID and count of every nonzero counter at its ascending rank r
// (out_ids[r], out_vals[r], only for r < lim) and clears every nonzero
// counter, whatever its rank.  Without offs, a block sums the counts of the
// blocks before it itself and the last one writes the totals: a launch less,
// and at most four loads a thread while nblk <= kDirectBlocks.
constexpr uint32_t kDirectBlocks = 1024;
__global__ void __launch_bounds__(256) k_req_write(uint32_t *__restrict__ cnt, uint64_t n,
                                                   const uint32_t *__restrict__ offs,
                                                   const uint32_t *__restrict__ blk,
                                                   const unsigned long long *__restrict__ sums,
                                                   CompactTotals *__restrict__ out, VolGeo g,
                                                   uint32_t *__restrict__ out_ids, uint32_t *__restrict__ out_vals,
                                                   uint32_t lim) {
    __shared__ uint32_t lds[4];
    __shared__ unsigned long long lds8[4];
    const uint64_t base = (uint64_t)blockIdx.x * 1024 + threadIdx.x * 4;
    const uint4 q = load_four(cnt, base, n);
    const uint32_t v[4] = {q.x, q.y, q.z, q.w};
    const uint32_t nz = (v[0] != 0) + (v[1] != 0) + (v[2] != 0) + (v[3] != 0);
    uint32_t before;
    const bool last = !offs && blockIdx.x == gridDim.x - 1;
    unsigned long long sum = 0;
    if (offs) {
        before = offs[blockIdx.x];
    } else {
        uint32_t a = 0;
        for (uint32_t b = threadIdx.x; b < blockIdx.x; b += 256) a += blk[b];
        before = (uint32_t)block_sum_256(a, lds8);
        if (last) {
            for (uint32_t b = threadIdx.x; b < gridDim.x; b += 256) sum += sums[b];
            sum = block_sum_256(sum, lds8);
        }
    }
    uint32_t tot;
    uint32_t r = before + block_excl_scan_256(nz, lds, &tot);
    if (last && threadIdx.x == 0) *out = {sum, before + tot, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (v[k]) {
            if (r < lim) {
                out_ids[r] = dense_to_id(g, (uint32_t)(base + k));
                out_vals[r] = v[k];
            }
            cnt[base + k] = 0;
            ++r;
        }
    }
}

ro_status read_requests_device(ro_cache *c, uint32_t cap, uint32_t *ids, uint32_t *counts,
                               uint32_t *n_unique, uint64_t *total, hipStream_t s) {
    return compact_dense(c, c->b.counters, cap, ids, counts, n_unique, total, s);
}

// Work space of one compaction of n entries: the totals, nblk = ceil(n /
// 1024) block counts and nblk + 1 offsets, nblk 64-bit block sums, and lim
// output IDs and values.
static constexpr uint64_t up256(uint64_t v) { return (v + 255) / 256 * 256; }

static constexpr uint64_t compact_bytes(uint64_t n, uint64_t lim) {
    const uint64_t nblk = (n + 1023) / 1024;
    return 256 + up256((2 * nblk + 1) * 4) + up256(nblk * 8) + 2 * up256(lim * 4);
}

size_t compact_scratch_bytes(uint64_t n, uint32_t lim) { return compact_bytes(n, lim); }

// Compaction of the dense per-brick array arr (g.total entries) in the work
// space ws (compact_scratch_bytes(g.total, lim) bytes, 256-byte aligned):
// copies the first min(cap, lim) (ID, value) pairs in ascending ID order to
// the host, with the distinct count and the sum, and clears the array.
// Synchronises.
ro_status compact_dense_ws(const VolGeo &g, uint32_t *arr, uint8_t *ws, uint32_t lim, uint32_t cap, uint32_t *ids,
                           uint32_t *counts, uint32_t *n_unique, uint64_t *total, hipStream_t s) {
    const uint32_t nblk = (uint32_t)((g.total + 1023) / 1024);
    CompactTotals *tot = (CompactTotals *)ws;
    uint32_t *blk = (uint32_t *)(ws + 256);
    uint32_t *offs = blk + nblk;
    unsigned long long *sums = (unsigned long long *)(ws + 256 + up256((2 * (uint64_t)nblk + 1) * 4));
    uint32_t *out_ids = (uint32_t *)((uint8_t *)sums + up256((uint64_t)nblk * 8));
    uint32_t *out_vals = out_ids + up256((uint64_t)lim * 4) / 4;
    hipLaunchKernelGGL(k_req_count, dim3(nblk), dim3(256), 0, s, arr, g.total, blk, sums);
    RO_HIP(hipGetLastError());
    const bool direct = nblk <= kDirectBlocks;
    if (!direct) {
        hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(256), 0, s, blk, nblk, offs, sums, tot);
        RO_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_req_write, dim3(nblk), dim3(256), 0, s, arr, g.total, direct ? nullptr : offs, blk, sums, tot,
                       g, out_ids, out_vals, lim);
    RO_HIP(hipGetLastError());
    CompactTotals t;
    RO_HIP(hipMemcpyAsync(&t, tot, sizeof(t), hipMemcpyDeviceToHost, s));
    RO_HIP(hipStreamSynchronize(s));
    uint32_t k = t.n < cap ? t.n : cap;
    k = k < lim ? k : lim;
    if (k) {
        RO_HIP(hipMemcpyAsync(ids, out_ids, 4 * (size_t)k, hipMemcpyDeviceToHost, s));
        RO_HIP(hipMemcpyAsync(counts, out_vals, 4 * (size_t)k, hipMemcpyDeviceToHost, s));
        RO_HIP(hipStreamSynchronize(s));
    }
    *n_unique = t.n;
    *total = t.sum;
    return RO_OK;
}

// Compaction in the cache's own scratch buffer (room for every brick).
ro_status compact_dense(ro_cache *c, uint32_t *arr, uint32_t cap, uint32_t *ids, uint32_t *counts,
                        uint32_t *n_unique, uint64_t *total, hipStream_t s) {
    const VolGeo &g = c->vol->g;
    return compact_dense_ws(g, arr, (uint8_t *)c->b.scratch + c->sc.compact, (uint32_t)g.total, cap, ids, counts,
                            n_unique, total, s);
}

// ------------------------------------- request readback without allocation

// Fixed work space of ro_read_requests_noalloc: room for the compaction of
// up to kNoAllocMaxBricks counters returning up to kNoAllocMaxPairs pairs.
// One copy per GPU, held until the process ends; every call on a GPU uses
// that GPU's copy, so calls that overlap on one GPU race.
constexpr uint64_t kNoAllocMaxBricks = 1ull << 26;
constexpr uint32_t kNoAllocMaxPairs = RO_NOALLOC_MAX_PAIRS;
constexpr size_t kNoAllocBytes = compact_bytes(kNoAllocMaxBricks, kNoAllocMaxPairs);

}  // namespace ro

static __device__ __align__(256) uint8_t scratch[ro::kNoAllocBytes];

namespace ro {

// Device address of this GPU's copy of `scratch` (the host-side name is not
// a device address): taken once per device with that device current.
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices];

static ro_status noalloc_scratch(uint8_t **out) {
    int dev = -1;
    RO_HIP(hipGetDevice(&dev));
    RO_CHECK(dev >= 0 && dev < kMaxDevices, RO_E_DEVICE, "device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        RO_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        RO_CHECK(p != nullptr, RO_E_DEVICE, "no device address for the fixed work space");
        g_scratch_ptr[dev] = p;
    }
    *out = (uint8_t *)g_scratch_ptr[dev];
    return RO_OK;
}

ro_status read_requests_noalloc_device(ro_cache *c, uint32_t cap, uint32_t *ids, uint32_t *counts,
                                       uint32_t *n_unique, uint64_t *total, hipStream_t s) {
    const VolGeo &g = c->vol->g;
    RO_CHECK(g.total <= kNoAllocMaxBricks, RO_E_CAPACITY,
             "volume has %llu bricks; the fixed work space holds counters of at most %llu",
             (unsigned long long)g.total, (unsigned long long)kNoAllocMaxBricks);
    RO_CHECK(cap <= kNoAllocMaxPairs, RO_E_CAPACITY, "cap %u exceeds the fixed work space's %u pairs", cap,
             kNoAllocMaxPairs);
    uint8_t *ws = nullptr;
    ro_status st = noalloc_scratch(&ws);
    if (st) return st;
    return compact_dense_ws(g, c->b.counters, ws, kNoAllocMaxPairs, cap, ids, counts, n_unique, total, s);
}

// -------------------------------------------------------- usage readback

__global__ void __launch_bounds__(256) k_use_count(const uint32_t *__restrict__ stamp,
                                                   const uint32_t *__restrict__ slot_brick, uint32_t n,
                                                   uint32_t f, uint32_t *__restrict__ blk) {
    __shared__ uint32_t lds[4];
    uint32_t base = blockIdx.x * 1024 + threadIdx.x * 4, nz = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) nz += (base + k < n) && stamp[base + k] == f && slot_brick[base + k] != kInvalid;
    uint32_t tot;
    block_excl_scan_256(nz, lds, &tot);
    if (threadIdx.x == 0) blk[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(256) k_use_write(const uint32_t *__restrict__ stamp,
                                                   const uint32_t *__restrict__ slot_brick, uint32_t n,
                                                   uint32_t f, const uint32_t *__restrict__ offs,
                                                   uint32_t *__restrict__ out) {
    __shared__ uint32_t lds[4];
    uint32_t base = blockIdx.x * 1024 + threadIdx.x * 4, nz = 0;
    bool hit[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        hit[k] = (base + k < n) && stamp[base + k] == f && slot_brick[base + k] != kInvalid;
        nz += hit[k];
    }
    uint32_t tot;
    uint32_t r = offs[blockIdx.x] + block_excl_scan_256(nz, lds, &tot);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (hit[k]) out[r++] = base + k;
}

ro_status read_usage_device(ro_cache *c, uint32_t frame, uint32_t cap, uint32_t *slots,
                            uint32_t *n_out, hipStream_t s) {
    uint8_t *sc = (uint8_t *)c->b.scratch;
    uint32_t S = c->desc.n_slots;
    uint32_t nblk = (S + 1023) / 1024;
    // the request-compaction block arrays are large enough: total >= 1 brick
    // per slot is not guaranteed, so use the candidate-key area when needed
    uint32_t *blk = (uint32_t *)(sc + c->sc.keys);  // n_slots * 8 bytes >= 2 * nblk + 1 words
    uint32_t *offs = blk + nblk + 1;
    uint32_t *out = (uint32_t *)(sc + c->sc.outpairs);
    hipLaunchKernelGGL(k_use_count, dim3(nblk), dim3(256), 0, s, c->b.stamps, c->b.slot_brick, S, frame, blk);
    RO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(256), 0, s, blk, nblk, offs,
                       (const unsigned long long *)nullptr, (CompactTotals *)nullptr);
    RO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_use_write, dim3(nblk), dim3(256), 0, s, c->b.stamps, c->b.slot_brick, S, frame,
                       offs, out);
    RO_HIP(hipGetLastError());
    uint32_t n = 0;
    RO_HIP(hipMemcpyAsync(&n, offs + nblk, 4, hipMemcpyDeviceToHost, s));
    RO_HIP(hipStreamSynchronize(s));
    uint32_t k = n < cap ? n : cap;
    if (k) {
        RO_HIP(hipMemcpyAsync(slots, out, 4 * (size_t)k, hipMemcpyDeviceToHost, s));
        RO_HIP(hipStreamSynchronize(s));
    }
    *n_out = n;
    return RO_OK;
}

// ------------------------------------------------------- LRU slot choice
//
// Radix select of the k smallest LRU keys, then their order by rank.  The
// time is launches and dependent round trips, not bytes: 218551 slots are
// 4 MB.  A slot's key has 64 bits but few of them differ within one cache
// (few frames are alive, and their sequence numbers lie close), so the keys
// pass reduces the ranges of the high and of the low words, and the digits
// are taken from (hi - hi_min) : (lo - lo_min), 11 bits each: three passes
// take 33 bits, where eight passes of a histogram and a pick took 64.  No
// block waits for another and none ends a pass for the others (a fence of
// device scope writes the XCD's L2 back: 38 us a pass): every block of the
// next launch picks the digit itself from the 2048 counts.  What the three
// passes leave undecided goes to the rank, if it is at most kSelSlack
// candidates more than asked for; if it is more, the collecting blocks count
// the further digits each for itself.

constexpr int kSelDigit = 11, kSelBins = 1 << kSelDigit, kSelPasses = 3;
constexpr uint32_t kSelThreads = 1024, kSelBlocks = 128;
static_assert(kSelHistWords == kSelPasses * kSelBins, "histogram area");
static_assert(kSelBins == 2 * kSelThreads, "two bins per thread");

// Choice after a pass: `krem` smallest of the keys whose short key equals
// `prefix` above bit `shift`, and all below; `extra` keys of the prefix are
// beyond those asked for.
struct SelChoice {
    unsigned long long prefix;
    uint32_t shift, krem, extra;
};

// Eligible slots and the ranges of their keys' high and low words.
struct SelRange {
    uint32_t elig, hmin, hmax, lmin, lmax, pad[3];
};
constexpr uint32_t kSelParts = 8;

// Select state (zero at the start but the minima, which are ~0).
struct SelState {
    uint32_t keff;          // min(eligible, asked for)
    uint32_t ncand;         // candidates collected
    uint32_t pad[2];
    SelChoice after[kSelPasses];  // [p]: the choice after pass p
    // of the blocks k, k + 8, ..: one part for all had 640 atomics queue for
    // one line (k_keys 12.6 us for 218551 slots)
    SelRange part[kSelParts];
};
static_assert(sizeof(SelState) <= 4 * kSelStateWords, "select state area");

// Key with the bits that no key of the cache uses taken out (the same order).
struct ShortKey {
    uint32_t hmin, lmin, lobits, bits, elig;
    __device__ ShortKey(const SelState *st) {
        uint32_t hmax = 0, lmax = 0;
        hmin = lmin = ~0u;
        elig = 0;
#pragma unroll
        for (uint32_t k = 0; k < kSelParts; ++k) {
            const SelRange r = st->part[k];
            elig += r.elig;
            hmin = min(hmin, r.hmin);
            hmax = max(hmax, r.hmax);
            lmin = min(lmin, r.lmin);
            lmax = max(lmax, r.lmax);
        }
        const uint32_t hr = hmax - hmin, lr = lmax - lmin;
        lobits = lr ? 32 - (uint32_t)__clz(lr) : 0;
        bits = lobits + (hr ? 32 - (uint32_t)__clz(hr) : 0);
    }
    __device__ unsigned long long operator()(unsigned long long k) const {
        return ((unsigned long long)((uint32_t)(k >> 32) - hmin) << lobits) | ((uint32_t)k - lmin);
    }
};

__device__ inline unsigned long long above(unsigned long long k, uint32_t shift) { return shift >= 64 ? 0 : k >> shift; }

// The choice before the first pass.
__device__ inline SelChoice sel_first(const ShortKey &sk, uint32_t n_new) {
    const uint32_t k = min(sk.elig, n_new);
    return {0, sk.bits, k, sk.elig - k};
}

// Next digit of a choice: its low bit and its mask.
__device__ inline uint32_t digit_shift(uint32_t shift) { return shift > kSelDigit ? shift - kSelDigit : 0; }
__device__ inline uint32_t digit_mask(uint32_t shift) { return (1u << (shift - digit_shift(shift))) - 1; }

// The choice after the digit of c, whose bins hold hist[] keys: the bin with
// the krem-th key.  By a whole block of 1024; every thread gets it.
__device__ inline SelChoice sel_pick(const SelChoice &c, const uint32_t *hist, SelChoice *lds, uint32_t *wsum) {
    const uint32_t b = 2 * threadIdx.x, v0 = hist[b], v1 = hist[b + 1];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t x = v0 + v1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wid] = x;
    if (threadIdx.x == 0) *lds = c;  // nothing to choose: krem is 0
    __syncthreads();
    uint32_t before = x - v0 - v1;
    for (int w = 0; w < wid; ++w) before += wsum[w];
    const uint32_t shift = digit_shift(c.shift);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t v = j ? v1 : v0;
        if (before < c.krem && c.krem <= before + v)  // one bin of the block
            *lds = {c.prefix | ((unsigned long long)(b + j) << shift), shift, c.krem - before,
                    before + v - c.krem};
        before += v;
    }
    __syncthreads();
    const SelChoice r = *lds;
    __syncthreads();
    return r;
}

// Counts the next digit of c over the block's share of the keys (from i0 on
// at the given stride) in h.  Between two barriers of the caller.
__device__ inline void sel_count(const SelChoice &c, const ShortKey &sk, const unsigned long long *__restrict__ keys,
                                 uint32_t S, uint32_t i0, uint32_t stride, uint32_t *h) {
    const uint32_t shift = digit_shift(c.shift), mask = digit_mask(c.shift);
    for (uint32_t i = i0 + threadIdx.x; i < S; i += stride) {
        const unsigned long long raw = keys[i];
        if (raw == ~0ull) continue;
        const unsigned long long k = sk(raw);
        if (above(k, c.shift) == above(c.prefix, c.shift)) atomicAdd(&h[(uint32_t)(k >> shift) & mask], 1u);
    }
}

// Stamps the resident bricks of the batch, and clears the histograms and the
// select state (a kernel, so that no memset stands between the launches).
__global__ void __launch_bounds__(1024) k_touch_clear(uint32_t *__restrict__ stamp, const uint32_t *__restrict__ slots,
                                                      uint32_t n, uint32_t f, uint32_t *__restrict__ hist,
                                                      SelState *__restrict__ st) {
    const uint32_t i = blockIdx.x * 1024 + threadIdx.x;
    if (i < n) stamp[slots[i]] = f;
    if (i < kSelHistWords) hist[i] = 0;
    if (i < kSelStateWords) ((uint32_t *)st)[i] = 0;
    __syncthreads();
    if (i < kSelParts) st->part[i].hmin = st->part[i].lmin = ~0u;
}

// LRU key per slot: free slots first in ascending index (key = slot), then
// occupied slots by (stamp, seq) (key = (stamp + 1) << 32 | seq); slots used
// in the current frame are not eligible (key = ~0).  Keys are unique.
__global__ void __launch_bounds__(1024) k_keys(const uint32_t *__restrict__ slot_brick,
                                               const uint32_t *__restrict__ stamp,
                                               const uint32_t *__restrict__ seq, uint32_t S, uint32_t f,
                                               unsigned long long *__restrict__ keys, SelState *__restrict__ state) {
    __shared__ uint32_t red[5];
    if (threadIdx.x < 5) red[threadIdx.x] = threadIdx.x == 1 || threadIdx.x == 3 ? ~0u : 0u;
    __syncthreads();
    uint32_t elig = 0, hmin = ~0u, hmax = 0, lmin = ~0u, lmax = 0;
    for (uint32_t i = blockIdx.x * kSelThreads + threadIdx.x; i < S; i += gridDim.x * kSelThreads) {
        const uint32_t sb = slot_brick[i], st = stamp[i], sq = seq[i];
        unsigned long long k = ((unsigned long long)(st + 1u) << 32) | sq;
        if (sb == kInvalid) k = i;
        else if (st == f) k = ~0ull;
        keys[i] = k;
        if (k != ~0ull) {
            ++elig;
            hmin = min(hmin, (uint32_t)(k >> 32));
            hmax = max(hmax, (uint32_t)(k >> 32));
            lmin = min(lmin, (uint32_t)k);
            lmax = max(lmax, (uint32_t)k);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        elig += __shfl_xor(elig, o, 64);
        hmin = min(hmin, (uint32_t)__shfl_xor(hmin, o, 64));
        hmax = max(hmax, (uint32_t)__shfl_xor(hmax, o, 64));
        lmin = min(lmin, (uint32_t)__shfl_xor(lmin, o, 64));
        lmax = max(lmax, (uint32_t)__shfl_xor(lmax, o, 64));
    }
    if ((threadIdx.x & 63) == 0 && elig) {
        atomicAdd(&red[0], elig);
        atomicMin(&red[1], hmin);
        atomicMax(&red[2], hmax);
        atomicMin(&red[3], lmin);
        atomicMax(&red[4], lmax);
    }
    __syncthreads();
    if (threadIdx.x == 0 && red[0]) {
        SelRange &part = state->part[blockIdx.x % kSelParts];
        atomicAdd(&part.elig, red[0]);
        atomicMin(&part.hmin, red[1]);
        atomicMax(&part.hmax, red[2]);
        atomicMin(&part.lmin, red[3]);
        atomicMax(&part.lmax, red[4]);
    }
}

// Choice before pass `pass`, the same in every thread (block 0 keeps it for
// the next launch).  done: no further digit is needed.
__device__ inline SelChoice sel_before(int pass, SelState *st, const ShortKey &sk, const uint32_t *hist,
                                       uint32_t n_new, SelChoice *lds, uint32_t *wsum) {
    if (pass == 0) return sel_first(sk, n_new);
    SelChoice c = pass == 1 ? sel_first(sk, n_new) : st->after[pass - 2];
    if (c.extra > 0 && c.krem > 0) c = sel_pick(c, hist + (pass - 1) * kSelBins, lds, wsum);
    if (blockIdx.x == 0 && threadIdx.x == 0) st->after[pass - 1] = c;
    return c;
}

// Pass 0, 1 or 2 of the select: histogram of the next digit over the keys of
// the prefix chosen so far.
__global__ void __launch_bounds__(1024) k_select(const unsigned long long *__restrict__ keys, uint32_t S,
                                                 SelState *state, uint32_t *__restrict__ hist, uint32_t n_new,
                                                 int pass) {
    __shared__ uint32_t h[kSelBins], wsum[kSelThreads / 64];
    __shared__ SelChoice lds;
    const ShortKey sk(state);
    const SelChoice c = sel_before(pass, state, sk, hist, n_new, &lds, wsum);
    if (c.extra == 0 || c.krem == 0) return;  // the prefix stands
    h[threadIdx.x] = 0;
    h[threadIdx.x + kSelThreads] = 0;
    __syncthreads();
    sel_count(c, sk, keys, S, blockIdx.x * kSelThreads, gridDim.x * kSelThreads, h);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t b = threadIdx.x + j * kSelThreads;
        if (h[b]) atomicAdd(&hist[pass * kSelBins + b], h[b]);
    }
}

// Collect the keys up to the end of the chosen prefix: at least the k_eff
// smallest, at most k_eff + kSelSlack.
__global__ void __launch_bounds__(1024) k_collect(const unsigned long long *__restrict__ keys, uint32_t S,
                                                  SelState *state, const uint32_t *__restrict__ hist, uint32_t n_new,
                                                  unsigned long long *__restrict__ cand,
                                                  uint32_t *__restrict__ cand_slot, uint32_t cap, int passes) {
    __shared__ uint32_t h[kSelBins], wsum[kSelThreads / 64];
    __shared__ SelChoice lds;
    const ShortKey sk(state);
    const uint32_t keff = min(sk.elig, n_new);
    if (blockIdx.x == 0 && threadIdx.x == 0) state->keff = keff;
    if (keff == 0) return;
    SelChoice c = sel_before(passes, state, sk, hist, n_new, &lds, wsum);
    while (c.extra > kSelSlack) {  // every block over all keys; a digit less each time, keys are unique
        h[threadIdx.x] = 0;
        h[threadIdx.x + kSelThreads] = 0;
        __syncthreads();
        sel_count(c, sk, keys, S, 0, kSelThreads, h);
        __syncthreads();
        const uint32_t left = c.shift;
        c = sel_pick(c, h, &lds, wsum);
        if (c.shift >= left) break;  // never with unique keys
    }
    const unsigned long long thr = above(c.prefix, c.shift);
    const int lane = threadIdx.x & 63;
    for (uint32_t i0 = blockIdx.x * kSelThreads; i0 < S; i0 += gridDim.x * kSelThreads) {
        const uint32_t i = i0 + threadIdx.x;
        const unsigned long long raw = i < S ? keys[i] : ~0ull;
        const bool in = raw != ~0ull && above(sk(raw), c.shift) <= thr;
        const unsigned long long bal = __ballot(in);
        if (bal == 0) continue;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&state->ncand, (uint32_t)__popcll(bal));
        at = __shfl(at, 0, 64) + (uint32_t)__popcll(bal & ((1ull << lane) - 1));
        if (in && at < cap) {
            cand[at] = raw;
            cand_slot[at] = i;
        }
    }
}

// Order of the candidates (rank = number of smaller keys; keys are unique)
// and the page-table update of the first k_eff: evict the victim's brick,
// insert the upload.  A wave ranks eight candidates, its lanes over all the
// others, so that 4096 candidates are 512 waves of 64 steps (one thread per
// candidate was 8 blocks of 2048 dependent LDS reads: 33 us for 2048).
constexpr uint32_t kRankPerWave = 8;
__global__ void __launch_bounds__(256) k_rank_update(const unsigned long long *__restrict__ cand,
                                                     const uint32_t *__restrict__ cand_slot,
                                                     const SelState *__restrict__ state, uint32_t cap,
                                                     const uint32_t *__restrict__ uploads,
                                                     uint32_t *__restrict__ victims, uint32_t *__restrict__ pt,
                                                     uint32_t *__restrict__ slot_brick,
                                                     uint32_t *__restrict__ stamp, uint32_t *__restrict__ seq,
                                                     uint32_t f, uint32_t seq_base) {
    const uint32_t k_eff = state->keff, n = min(state->ncand, cap);
    const uint32_t i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kRankPerWave;
    const uint32_t lane = threadIdx.x & 63;
    if (k_eff == 0 || i0 >= n) return;
    const unsigned long long own = i0 + (lane & 7) < n ? cand[i0 + (lane & 7)] : 0;
    unsigned long long mine[kRankPerWave];
    uint32_t cnt[kRankPerWave];
#pragma unroll
    for (uint32_t r = 0; r < kRankPerWave; ++r) {
        mine[r] = __shfl(own, (int)r, 64);
        cnt[r] = 0;
    }
    for (uint32_t j0 = 0; j0 < n; j0 += 512) {  // eight loads in flight
        unsigned long long o[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
            const uint32_t j = j0 + 64 * q + lane;
            o[q] = cand[min(j, n - 1)];
            if (j >= n) o[q] = ~0ull;
        }
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q)
#pragma unroll
            for (uint32_t r = 0; r < kRankPerWave; ++r) cnt[r] += (uint32_t)__popcll(__ballot(o[q] < mine[r]));
    }
    uint32_t rank = 0;
#pragma unroll
    for (uint32_t r = 0; r < kRankPerWave; ++r) rank = lane == r ? cnt[r] : rank;
    if (lane >= kRankPerWave || i0 + lane >= n || rank >= k_eff) return;
    const uint32_t slot = cand_slot[i0 + lane], old = slot_brick[slot], b = uploads[rank];
    if (old != kInvalid) pt[old] = kInvalid;
    victims[rank] = slot;
    pt[b] = slot;
    slot_brick[slot] = b;
    stamp[slot] = f;
    seq[slot] = seq_base + rank;
}

// Brick scatter: staged brick src[i] -> slot victims[i], 16-byte vectors.
__global__ void __launch_bounds__(256) k_scatter(const SelState *__restrict__ state,
                                                 const uint32_t *__restrict__ victims,
                                                 const uint32_t *__restrict__ src,
                                                 const uint4 *__restrict__ staged, uint4 *__restrict__ slots,
                                                 uint32_t vec_per_slot) {
    uint32_t i = blockIdx.y;
    if (i >= state->keff) return;
    const uint4 *from = staged + (size_t)src[i] * vec_per_slot;
    uint4 *to = slots + (size_t)victims[i] * vec_per_slot;
    for (uint32_t v = blockIdx.x * 256 + threadIdx.x; v < vec_per_slot; v += gridDim.x * 256)
        to[v] = from[v];
}

ro_status stream_bricks_device(ro_cache *c, uint32_t frame, uint32_t n_new, uint32_t n_touch,
                               const void *staged, hipStream_t s, uint32_t *result) {
    const VolGeo &g = c->vol->g;
    uint8_t *sc = (uint8_t *)c->b.scratch;
    const uint32_t S = c->desc.n_slots;
    unsigned long long *keys = (unsigned long long *)(sc + c->sc.keys);
    uint32_t *hist = (uint32_t *)(sc + c->sc.hist);
    SelState *sel = (SelState *)(sc + c->sc.sel);
    unsigned long long *cand = (unsigned long long *)(sc + c->sc.cand);
    uint32_t *victims = (uint32_t *)sel + kSelStateWords;  // read back with the state in one copy
    const uint32_t *uploads = (uint32_t *)(sc + c->sc.batch), *srcidx = uploads + n_new, *touch = srcidx + n_new;
    uint32_t *cand_slot = (uint32_t *)(sc + c->sc.outpairs);  // at least n_slots words
    if (n_new + n_touch == 0) return RO_OK;
    ro_status st = c->batch.send(sc + c->sc.batch);
    if (st) return st;
    hipLaunchKernelGGL(k_touch_clear, dim3((std::max(n_touch, kSelHistWords) + 1023) / 1024), dim3(1024), 0, s,
                       c->b.stamps, touch, n_touch, frame, hist, sel);
    RO_HIP(hipGetLastError());
    if (n_new == 0) {
        c->batch.mark();
        return RO_OK;
    }
    const uint32_t cap = std::min(n_new + kSelSlack, S);
    const uint32_t nb = std::min((S + kSelThreads - 1) / kSelThreads, kSelBlocks);
    // no pass where all slots fit the candidates: the rank takes them apart
    const int passes = S > cap ? kSelPasses : 0;
    hipLaunchKernelGGL(k_keys, dim3(nb), dim3(kSelThreads), 0, s, c->b.slot_brick, c->b.stamps, c->b.seqs, S, frame,
                       keys, sel);
    RO_HIP(hipGetLastError());
    for (int p = 0; p < passes; ++p) {
        hipLaunchKernelGGL(k_select, dim3(nb), dim3(kSelThreads), 0, s, keys, S, sel, hist, n_new, p);
        RO_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_collect, dim3(nb), dim3(kSelThreads), 0, s, keys, S, sel, hist, n_new, cand, cand_slot, cap,
                       passes);
    RO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_rank_update, dim3((cap + 4 * kRankPerWave - 1) / (4 * kRankPerWave)), dim3(256), 0, s, cand,
                       cand_slot, sel, cap, uploads, victims, c->b.page_table, c->b.slot_brick, c->b.stamps,
                       c->b.seqs, frame, c->seq_next);
    RO_HIP(hipGetLastError());
    uint32_t vps = g.slot_stride / 16;
    uint32_t gx = (vps + 255) / 256;
    hipLaunchKernelGGL(k_scatter, dim3(gx, n_new), dim3(256), 0, s, sel, victims, srcidx,
                       (const uint4 *)staged, (uint4 *)c->b.slots, vps);
    RO_HIP(hipGetLastError());
    RO_HIP(hipMemcpyAsync(result, sel, 4 * (kSelStateWords + (size_t)n_new), hipMemcpyDeviceToHost, s));
    RO_HIP(hipStreamSynchronize(s));
    c->batch.done();
    result[0] = ((const SelState *)result)->keff;
    memmove(result + 1, result + kSelStateWords, 4 * (size_t)result[0]);
    return RO_OK;
}

// Every resident brick whose dense index lies in [lo, hi) leaves the cache:
// its page-table entry and its slot's brick are cleared, so the slot is free.
__global__ void k_evict_range(uint32_t *__restrict__ slot_brick, uint32_t *__restrict__ pt, uint32_t S,
                              uint32_t lo, uint32_t hi) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S) return;
    const uint32_t b = slot_brick[i];
    if (b != kInvalid && b >= lo && b < hi) {
        pt[b] = kInvalid;
        slot_brick[i] = kInvalid;
    }
}

ro_status cache_evict_channel(ro_cache *c, uint32_t ch, hipStream_t s) {
    const VolGeo &g = c->vol->g;
    const uint32_t lo = ch * g.per_channel, hi = lo + g.per_channel;
    const uint32_t S = c->desc.n_slots;
    hipLaunchKernelGGL(k_evict_range, dim3((S + 255) / 256), dim3(256), 0, s, c->b.slot_brick, c->b.page_table, S,
                       lo, hi);
    RO_HIP(hipGetLastError());
    // the host mirrors follow; the evicted bricks await the residency update
    for (uint32_t i = 0; i < S; ++i) {
        const uint32_t b = c->slot_host[i];
        if (b != kInvalid && b >= lo && b < hi) {
            c->pt_host[b] = kInvalid;
            c->slot_host[i] = kInvalid;
            c->dirty.push_back(b);
        }
    }
    return RO_OK;
}

}  // namespace ro
