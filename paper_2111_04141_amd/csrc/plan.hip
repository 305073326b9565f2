// Plan building: index rule, bucket counting sort, chunk list, per-chunk
// cell sort.
//
// The thesis sorts records by their position on the virtual NN grid before
// gridding ("SS" ordering, Section 3.2.4) because the order in which records
// reach the gridder sets how often accumulated values have to be committed
// (Chapter 4).  Here the order is (plane, uv tile, cell): a counting sort by
// (plane, tile) bucket over the whole record set, then a counting sort by
// cell inside each chunk of at most R records.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"

namespace mg {

namespace {

constexpr uint32_t kInvalidBucket = 0xffffffffu;

// ---------------------------------------------------------------------------
// index rule -> bucket histogram and skipped count; the scatter evaluates the
// rule again (reading uvw costs what storing and re-reading its results
// would, and saves writing them)
// ---------------------------------------------------------------------------
// Packed meta and bucket of record r (bucket kInvalidBucket if skipped).
template <typename T>
__device__ inline RecIndex index_bucket(const DevGeom &g, const PlaneLayout *planes,
                                        const T *uvw, int64_t r, uint32_t *bucket) {
    const RecIndex ix = index_record<T>(g, uvw[3 * r], uvw[3 * r + 1], uvw[3 * r + 2]);
    uint32_t b = kInvalidBucket;
    if (ix.valid) {
        const int p = ix.plane < 0 ? 0 : ix.plane;
        const PlaneLayout pl = planes[p];
        const uint32_t tu = (uint32_t)ix.ku >> pl.log2T;
        const uint32_t tv = (uint32_t)ix.kv >> pl.log2T;
        b = (uint32_t)(pl.base + ((int64_t)tv * pl.ntu + tu) * pl.grp_n + (p - pl.grp_first));
    }
    *bucket = b;
    return ix;
}

// The plan's tap table, phase-major (see common.h): entry
// (o_v, o_u, j, i) of plane p takes bank element (o_v + 1 + j beta) *
// (beta S + 1) + (o_u + 1 + i beta) of the caller's plane; for W-projection
// (complex entries, (re, im) pairs of T) its conjugate also goes to
// conj_base + the same index.  Separable: entry (o, i) takes o + 1 + i beta.
// Also raises planes[p].tmax to the largest |component| copied (the plane
// layouts arrive with tmax = 0; non-negative floats order like their bits).
// Workgroup `block` of `blocks` for plane p.
template <typename T>
__device__ inline void tap_layout(PlaneLayout *planes, int p, int block, int blocks, int32_t beta,
                                  int32_t wproj, const T *__restrict__ src, T *__restrict__ dst,
                                  int64_t conj_base) {
    const PlaneLayout pl = planes[p];
    const int64_t S = pl.S;
    const int64_t ws = (int64_t)beta * S + 1;   // caller's row length
    const int64_t n = wproj ? (int64_t)beta * beta * S * S : (int64_t)beta * S;
    float m = 0.0f;
    for (int64_t e = (int64_t)block * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)blocks * blockDim.x) {
        const int64_t i = e % S;
        const int64_t d = (int64_t)pl.tap_off + e;
        if (wproj) {
            const int64_t blk = e / (S * S);
            const int64_t j = (e / S) % S;
            const int64_t ou = blk % beta, ov = blk / beta;
            const int64_t sidx = (int64_t)pl.src_off + (ov + 1 + j * beta) * ws + (ou + 1 + i * beta);
            const T re = src[2 * sidx], im = src[2 * sidx + 1];
            dst[2 * d] = re;
            dst[2 * d + 1] = im;
            dst[2 * (conj_base + d)] = re;
            dst[2 * (conj_base + d) + 1] = -im;
            m = fmaxf(m, fmaxf(fabsf(TapTraits<T>::real(&re, 0)), fabsf(TapTraits<T>::real(&im, 0))));
        } else {
            const int64_t o = e / S;
            const T t = src[o + 1 + i * beta];
            dst[d] = t;
            m = fmaxf(m, fabsf(TapTraits<T>::real(&t, 0)));
        }
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0 && m > 0.0f)
        atomicMax(reinterpret_cast<unsigned int *>(&planes[p].tmax), __float_as_uint(m));
}

// Calls of few buckets (kLdsBuckets: grids up to 1448^2 of one plane, the
// smallest calls, bound by latency) count in LDS first: a counter of a dense
// tile takes an atomic about every 10 ns, so 100,800 one-channel records on 4096
// tiles, few lanes of a wave sharing one, took 22 us here and 24 us in the
// scatter.  A workgroup takes kLdsRecords consecutive records (and clears and
// reads every counter: beyond a million records the aggregated atomics of a
// wave are left the cheaper way).
constexpr int64_t kLdsBuckets = 8192;
constexpr int kLdsPerThread = 4;
constexpr int kLdsRecords = 256 * kLdsPerThread;
constexpr int64_t kLdsCallRecords = 1024 * (int64_t)kLdsRecords;

// The plane layouts a plan is built with (kernel argument: up to kPlaneArgs a
// launch, below the argument limit), and the words that start at zero.
constexpr int kPlaneArgs = 56;
struct PlaneArgs {
    PlaneLayout pl[kPlaneArgs];
};

__global__ __launch_bounds__(256) void setup_kernel(PlaneArgs a, int32_t p0, int32_t n,
                                                    PlaneLayout *__restrict__ planes,
                                                    int64_t *__restrict__ counters,
                                                    uint32_t *__restrict__ group_nunits,
                                                    int32_t nplanes, uint32_t *__restrict__ hist,
                                                    int64_t nb) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0) {
        if ((int)threadIdx.x < n) planes[p0 + threadIdx.x] = a.pl[threadIdx.x];
        if (threadIdx.x < 6) counters[threadIdx.x] = 0;
        if ((int)threadIdx.x < nplanes) group_nunits[threadIdx.x] = 0u;
    }
    // (the arena is 256-byte aligned and its arrays padded to 256 bytes)
    uint4 *h = reinterpret_cast<uint4 *>(hist);
    for (int64_t i = i0; i < (nb + 3) / 4; i += (int64_t)gridDim.x * blockDim.x)
        h[i] = make_uint4(0u, 0u, 0u, 0u);
}

// The first `tap_blocks` workgroups lay out the tap table (tap_layout), the
// others count the records of every bucket and the skipped ones.
template <typename T, typename TapT, bool LDS>
__global__ __launch_bounds__(256) void index_taps_kernel(
    DevGeom g, PlaneLayout *planes, int64_t nrec, const T *__restrict__ uvw,
    uint32_t *__restrict__ hist, int32_t nb, int64_t *__restrict__ counters, int32_t tap_blocks,
    int32_t tap_per_plane, int32_t wproj, const TapT *__restrict__ src, TapT *__restrict__ dst,
    int64_t conj_base) {
    if ((int)blockIdx.x < tap_blocks) {
        tap_layout<TapT>(planes, blockIdx.x / tap_per_plane, blockIdx.x % tap_per_plane,
                         tap_per_plane, g.beta, wproj, src, dst, conj_base);
        return;
    }
    __shared__ uint32_t s_skip;
    extern __shared__ uint32_t s_hist[];
    if (threadIdx.x == 0) s_skip = 0;
    if constexpr (LDS)
        for (int i = threadIdx.x; i < nb; i += blockDim.x) s_hist[i] = 0u;
    __syncthreads();
    uint32_t skipped = 0;
    const int64_t block = (int64_t)blockIdx.x - tap_blocks, blocks = (int64_t)gridDim.x - tap_blocks;
    if constexpr (LDS) {
        for (int k = 0; k < kLdsPerThread; ++k) {
            const int64_t r = block * kLdsRecords + k * 256 + threadIdx.x;
            if (r >= nrec) break;
            uint32_t b;
            index_bucket<T>(g, planes, uvw, r, &b);
            if (b == kInvalidBucket)
                ++skipped;
            else
                atomicAdd(&s_hist[b], 1u);
        }
    } else {
        // every lane of a wave runs the same number of iterations (the
        // aggregated atomic needs the whole wave)
        const int64_t stride = blocks * blockDim.x;
        const int64_t first = block * blockDim.x + (threadIdx.x & ~63);
        for (int64_t r0 = first; r0 < nrec; r0 += stride) {
            const int64_t r = r0 + (threadIdx.x & 63);
            const bool in = r < nrec;
            uint32_t b = kInvalidBucket;
            if (in) index_bucket<T>(g, planes, uvw, r, &b);
            if (in && b == kInvalidBucket) ++skipped;
            wave_counter_add(hist, b, b != kInvalidBucket, false);
        }
    }
    if (skipped) atomicAdd(&s_skip, skipped);
    __syncthreads();
    if constexpr (LDS)
        for (int i = threadIdx.x; i < nb; i += blockDim.x)
            if (s_hist[i]) atomicAdd(&hist[i], s_hist[i]);
    if (threadIdx.x == 0 && s_skip) atomicAdd((unsigned long long *)&counters[0],
                                              (unsigned long long)s_skip);
}

// ---------------------------------------------------------------------------
// exclusive scan of (count, chunks-of-R) pairs over the buckets
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 1024;
constexpr int kScanItems = 4;
constexpr int kScanBlock = kScanThreads * kScanItems;
// Blocks whose sums every workgroup adds up for itself; more are scanned in a
// launch of their own.  Builds of 1000 records, added up and scanned: 4.2M
// buckets (1024 blocks) 103 us both, 67M 646 and 555 us, 1074M 26.1 and 8.3 ms.
constexpr int64_t kScanSums = 1024;

__device__ inline uint2 add2(uint2 a, uint2 b) { return make_uint2(a.x + b.x, a.y + b.y); }

// This thread's buckets' counts (0 past the end; hist is padded to 256 bytes).
__device__ inline uint4 counts_of(const uint32_t *hist, int64_t i, int64_t n) {
    uint4 c = make_uint4(0u, 0u, 0u, 0u);
    if (i < n) c = *reinterpret_cast<const uint4 *>(hist + i);
    if (i + 1 >= n) c.y = 0u;
    if (i + 2 >= n) c.z = 0u;
    if (i + 3 >= n) c.w = 0u;
    return c;
}
// (records, chunks of R) of four buckets
__device__ inline uint2 pair_of(uint4 c, uint32_t R) {
    return make_uint2(c.x + c.y + c.z + c.w,
                      (c.x + R - 1) / R + (c.y + R - 1) / R + (c.z + R - 1) / R + (c.w + R - 1) / R);
}

// Workgroup-wide exclusive scan of one pair per thread; *total: the sum.
__device__ inline uint2 block_exclusive_scan(uint2 v, uint2 *total) {
    __shared__ uint2 s[kScanThreads / kWave];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint2 incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t x = (uint32_t)__shfl_up((int)incl.x, d, 64);
        const uint32_t y = (uint32_t)__shfl_up((int)incl.y, d, 64);
        if (lane >= d) incl = add2(incl, make_uint2(x, y));
    }
    __syncthreads();
    if (lane == 63) s[wave] = incl;
    __syncthreads();
    uint2 before = make_uint2(0u, 0u), sum = make_uint2(0u, 0u);
    for (int w = 0; w < kScanThreads / kWave; ++w) {
        if (w < wave) before = add2(before, s[w]);
        sum = add2(sum, s[w]);
    }
    *total = sum;
    return make_uint2(before.x + incl.x - v.x, before.y + incl.y - v.y);
}

// Sums of the scan's blocks (calls of more than one block).
__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(
    const uint32_t *__restrict__ hist, int64_t n, uint32_t R, uint2 *__restrict__ block_sums) {
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
    uint2 total;
    block_exclusive_scan(pair_of(counts_of(hist, i, n), R), &total);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// Exclusive scan of the block sums, in place, by one workgroup.
__global__ __launch_bounds__(kScanThreads) void scan_sums_kernel(uint2 *__restrict__ sums,
                                                                 int64_t n) {
    uint2 carry = make_uint2(0u, 0u);
    for (int64_t first = 0; first < n; first += kScanBlock) {
        const int64_t i = first + (int64_t)threadIdx.x * kScanItems;
        uint2 v[kScanItems], mine = make_uint2(0u, 0u), total;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = i + k < n ? sums[i + k] : make_uint2(0u, 0u);
            mine = add2(mine, v[k]);
        }
        uint2 run = add2(carry, block_exclusive_scan(mine, &total));
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (i + k < n) sums[i + k] = run;
            run = add2(run, v[k]);
        }
        carry = add2(carry, total);
    }
}

// Writes cursor[i] (first record of bucket i, advanced by the scatter),
// cstart[i] (first chunk of bucket i) and the chunks: bucket b with c records
// -> ceil(c/R) chunks.  The sum of the blocks before a workgroup's own is
// block_sums[its number] where they have been scanned; else it adds them up.  Also plane_cfirst[p] = first
// chunk of plane p's group, plane_cfirst[P] = cstart[n] = counters[2] = chunk
// count, counters[1] = valid records (counters[3] counts the skipped records
// placed by the scatter).
__global__ __launch_bounds__(kScanThreads) void scan_chunks_kernel(
    const uint32_t *__restrict__ hist, int64_t n, uint32_t R,
    const uint2 *__restrict__ block_sums, int32_t scanned, uint32_t *__restrict__ cursor,
    uint32_t *__restrict__ cstart, Chunk *__restrict__ chunks,
    const PlaneLayout *__restrict__ planes, int32_t nplanes, uint32_t *__restrict__ plane_cfirst,
    int64_t *__restrict__ counters) {
    uint2 offset;
    if (scanned) {
        offset = block_sums[blockIdx.x];
    } else {
        uint2 mine = make_uint2(0u, 0u);
        for (int j = threadIdx.x; j < (int)blockIdx.x; j += kScanThreads)
            mine = add2(mine, block_sums[j]);
        block_exclusive_scan(mine, &offset);
    }
    const int64_t first = (int64_t)blockIdx.x * kScanBlock;
    const int64_t i = first + (int64_t)threadIdx.x * kScanItems;
    const uint4 c4 = counts_of(hist, i, n);
    uint2 total;
    uint2 run = add2(block_exclusive_scan(pair_of(c4, R), &total), offset);
    const uint32_t c[kScanItems] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (i + k < n) {
            cursor[i + k] = run.x;
            cstart[i + k] = run.y;
            for (uint32_t m = 0; m * R < c[k]; ++m) {
                Chunk ch;
                ch.start = run.x + m * R;
                ch.len = min(R, c[k] - m * R);
                ch.bucket = (uint32_t)(i + k);
                ch.bbox = 0;
                chunks[run.y + m] = ch;
            }
        }
        run = add2(run, make_uint2(c[k], (c[k] + R - 1) / R));
    }
    __syncthreads();   // (cstart of this block's buckets is read back)
    for (int p = threadIdx.x; p < nplanes; p += kScanThreads) {
        const int64_t b = planes[p].base;
        if (b >= first && b < first + kScanBlock && b < n) plane_cfirst[p] = cstart[b];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const uint2 all = add2(offset, total);
        plane_cfirst[nplanes] = all.y;
        cstart[n] = all.y;
        counters[1] = all.x;
        counters[2] = all.y;
    }
}

// ---------------------------------------------------------------------------
// scatter records into bucket order (order inside a bucket is arbitrary;
// the chunk sort below orders each chunk by cell)
// ---------------------------------------------------------------------------
// Valid records go to their bucket's slots; skipped records follow all valid
// ones (sperm only: their outputs are zeroed by the degridder).  LDS: the
// workgroup's records of each bucket are counted in LDS and take consecutive
// slots, one atomic per bucket (see index_taps_kernel).
template <typename T, bool LDS>
__global__ __launch_bounds__(256) void scatter_kernel(DevGeom g,
                                                      const PlaneLayout *__restrict__ planes,
                                                      int64_t nrec, const T *__restrict__ uvw,
                                                      uint32_t *__restrict__ cursor, int32_t nb,
                                                      int64_t *__restrict__ counters,
                                                      RecMeta *__restrict__ smeta,
                                                      uint32_t *__restrict__ sperm) {
    const int64_t nvalid = counters[1];
    auto skip = [&](int64_t r) {
        const int64_t q = nvalid + (int64_t)atomicAdd((unsigned long long *)&counters[3], 1ull);
        if (q < nrec) sperm[q] = (uint32_t)r;
    };
    if constexpr (LDS) {
        extern __shared__ uint32_t s_cnt[];
        for (int i = threadIdx.x; i < nb; i += blockDim.x) s_cnt[i] = 0u;
        __syncthreads();
        RecMeta m[kLdsPerThread];
        uint32_t b[kLdsPerThread], rank[kLdsPerThread];
#pragma unroll
        for (int k = 0; k < kLdsPerThread; ++k) {
            const int64_t r = (int64_t)blockIdx.x * kLdsRecords + k * 256 + threadIdx.x;
            b[k] = kInvalidBucket;
            if (r >= nrec) continue;
            const RecIndex ix = index_bucket<T>(g, planes, uvw, r, &b[k]);
            m[k] = pack_meta(g, ix);
            if (b[k] != kInvalidBucket)
                rank[k] = atomicAdd(&s_cnt[b[k]], 1u);
            else
                skip(r);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < nb; i += blockDim.x)
            if (s_cnt[i]) s_cnt[i] = atomicAdd(&cursor[i], s_cnt[i]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kLdsPerThread; ++k) {
            if (b[k] == kInvalidBucket) continue;
            const uint32_t pos = s_cnt[b[k]] + rank[k];
            smeta[pos] = m[k];
            sperm[pos] = (uint32_t)((int64_t)blockIdx.x * kLdsRecords + k * 256 + threadIdx.x);
        }
    } else {
        const int64_t stride = (int64_t)gridDim.x * blockDim.x;
        const int64_t first = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63);
        for (int64_t r0 = first; r0 < nrec; r0 += stride) {
            const int64_t r = r0 + (threadIdx.x & 63);
            uint32_t b = kInvalidBucket;
            RecIndex ix;
            if (r < nrec) ix = index_bucket<T>(g, planes, uvw, r, &b);
            const bool act = b != kInvalidBucket;
            const uint32_t pos = wave_counter_add(cursor, b, act, true);
            if (act) {
                smeta[pos] = pack_meta(g, ix);
                sperm[pos] = (uint32_t)r;
            } else if (r < nrec) {
                skip(r);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// units of a plane group: the chunks of one tile, over
// all planes of the group, split greedily into runs of at most `cap`
// records (a chunk is never split).  The gridders take a unit at a time
// and commit the tile's region once per unit rather than once per chunk.
// units[first chunk of the group + k] = (first chunk, chunk count) of the group's
// unit k; group_nunits[g] = unit count (cleared beforehand).
// A wave's units are consecutive and in tile order.
// A launch covers its groups (blockIdx.y) and every tile (a thread each).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void unit_list_kernel(const PlaneLayout *__restrict__ planes,
                                                        GroupList groups,
                                                        const uint32_t *__restrict__ bucket_cfirst,
                                                        const Chunk *__restrict__ chunks,
                                                        uint32_t cap, uint2 *__restrict__ units,
                                                        uint32_t *__restrict__ group_nunits) {
    const int g = groups.first[blockIdx.y];
    const PlaneLayout pl = planes[g];
    const uint32_t ntiles = (uint32_t)pl.ntu * (uint32_t)pl.ntv;
    const uint32_t n = (uint32_t)pl.grp_n;
    const int64_t base = pl.base;
    const int lane = threadIdx.x & 63;
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t cs = 0, ce = 0;
    if (t < ntiles) {
        cs = bucket_cfirst[base + (int64_t)t * n];
        ce = bucket_cfirst[base + (int64_t)(t + 1) * n];
    }
    // A bucket's chunks are full (cap records) but for its last one, so the
    // greedy split only has to look at each bucket's chunk count and last
    // length: full chunks are units of their own, and a bucket's last chunk
    // joins the open unit if it fits (acc = cap opens a unit at the first
    // chunk).
    auto walk = [&](auto emit) {
        uint32_t acc = cap, head = cs;
        for (uint32_t j = 0; j < n && cs < ce; ++j) {
            const int64_t b = base + (int64_t)t * n + j;
            const uint32_t b0 = bucket_cfirst[b], b1 = bucket_cfirst[b + 1];
            if (b0 == b1) continue;
            const uint32_t last_len = chunks[b1 - 1].len;
            for (uint32_t c = b0; c + 1 < b1; ++c) {   // full chunks
                if (c > head) emit(head, c);
                head = c;
                acc = cap;
            }
            if (acc + last_len > cap) {
                if (b1 - 1 > head) emit(head, b1 - 1);
                head = b1 - 1;
                acc = last_len;
            } else {
                acc += last_len;
            }
        }
        if (ce > cs) emit(head, ce);
    };
    // pass 1: unit count of this tile
    uint32_t cnt = 0;
    walk([&](uint32_t, uint32_t) { ++cnt; });
    // wave prefix sum; one lane reserves the wave's units
    uint32_t incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    const uint32_t wtotal = __shfl(incl, 63, 64);
    uint32_t wbase = 0;
    if (lane == 63 && wtotal) wbase = atomicAdd(&group_nunits[g], wtotal);
    wbase = __shfl(wbase, 63, 64);
    // pass 2: write them
    uint2 *out = units + bucket_cfirst[base] + wbase + (incl - cnt);
    walk([&](uint32_t h, uint32_t e) { *out++ = make_uint2(h, e - h); });
}

// ---------------------------------------------------------------------------
// per-chunk counting sort by cell inside the tile, in LDS: column by column
// (u outer), v running up and down in alternate columns, so consecutive
// records step by one cell and a moving window retires one row or column of
// slots at a time (a plain column-major order would retire most slots at
// every column change)
// ---------------------------------------------------------------------------
constexpr int kMaxR = 2048;

__device__ inline uint32_t cell_key(uint32_t du, uint32_t dv, int log2T) {
    const uint32_t vv = (du & 1u) ? ((1u << log2T) - 1u - dv) : dv;
    return (du << log2T) | vv;
}


// Chunks of at most kWaveSortMax records: one wave per chunk sorts the
// (cell key, lane) pairs with a bitonic network across its lanes, then each
// lane fetches the record of its rank; no LDS and no barriers.  Larger
// chunks take the workgroup counting sort below.
constexpr uint32_t kWaveSortMax = 64;

__device__ inline void sort_small_chunks(const uint32_t *__restrict__ plane_cfirst,
                                         int32_t nplanes, const PlaneLayout *__restrict__ planes,
                                         Chunk *__restrict__ chunks, RecMeta *__restrict__ smeta,
                                         uint32_t *__restrict__ sperm, uint32_t block,
                                         uint32_t blocks) {
    const uint32_t c_end = plane_cfirst[nplanes];
    const int lane = threadIdx.x & 63;
    const uint32_t nwaves = blocks * (blockDim.x >> 6);
    int p = 0;   // chunks come in increasing order: the plane only moves forward
    for (uint32_t c = block * (blockDim.x >> 6) + (threadIdx.x >> 6); c < c_end; c += nwaves) {
        const Chunk ch = chunks[c];
        if (ch.len > kWaveSortMax) continue;
        while (p + 1 < nplanes && c >= plane_cfirst[p + 1]) ++p;
        int pp;
        uint32_t tile;
        bucket_plane_tile(planes[p], ch.bucket, &pp, &tile);
        const PlaneLayout pl = planes[pp];
        if (pl.cls >= 3) continue;   // the blocked kernels need neither
        const uint32_t tu0 = (tile % (uint32_t)pl.ntu) << pl.log2T;
        const uint32_t tv0 = (tile / (uint32_t)pl.ntu) << pl.log2T;
        RecMeta m{0u, 0u};
        uint32_t perm = 0u;
        uint32_t v = 0xffffffffu;   // lanes past the chunk sort last
        uint32_t umin = 0xffu, umax = 0u, vmin = 0xffu, vmax = 0u;
        if ((uint32_t)lane < ch.len) {
            m = smeta[ch.start + lane];
            perm = sperm[ch.start + lane];
            const uint32_t du = meta_ku(m) - tu0, dv = meta_kv(m) - tv0;
            v = (cell_key(du, dv, pl.log2T) << 6) | (uint32_t)lane;
            umin = umax = du;
            vmin = vmax = dv;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            umin = min(umin, (uint32_t)__shfl_xor((int)umin, off, 64));
            umax = max(umax, (uint32_t)__shfl_xor((int)umax, off, 64));
            vmin = min(vmin, (uint32_t)__shfl_xor((int)vmin, off, 64));
            vmax = max(vmax, (uint32_t)__shfl_xor((int)vmax, off, 64));
        }
        if (lane == 0) chunks[c].bbox = umin | (umax << 8) | (vmin << 16) | (vmax << 24);
        if (ch.len < 2) continue;
#pragma unroll
        for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
                const uint32_t o = (uint32_t)__shfl_xor((int)v, j, 64);
                const bool take_min = ((lane & j) == 0) == ((lane & k) == 0);
                v = take_min ? min(v, o) : max(v, o);
            }
        }
        const int src = (int)(v & 63u);
        const uint32_t kuv = (uint32_t)__shfl((int)m.kuv, src, 64);
        const uint32_t toff = (uint32_t)__shfl((int)m.toff, src, 64);
        const uint32_t pr = (uint32_t)__shfl((int)perm, src, 64);
        if ((uint32_t)lane < ch.len) {
            smeta[ch.start + lane] = RecMeta{kuv, toff};
            sperm[ch.start + lane] = pr;
        }
    }
}

__global__ __launch_bounds__(256) void chunk_sort_kernel(const uint32_t *__restrict__ plane_cfirst,
                                                         int32_t nplanes,
                                                         const PlaneLayout *__restrict__ planes,
                                                         Chunk *__restrict__ chunks,
                                                         RecMeta *__restrict__ smeta,
                                                         uint32_t *__restrict__ sperm,
                                                         int32_t small_blocks) {
    // the first workgroups take the small chunks, a wave each
    if ((int)blockIdx.x < small_blocks) {
        sort_small_chunks(plane_cfirst, nplanes, planes, chunks, smeta, sperm, blockIdx.x,
                          (uint32_t)small_blocks);
        return;
    }
    __shared__ uint32_t hist[1024];
    __shared__ RecMeta m_in[kMaxR];
    __shared__ uint32_t p_in[kMaxR];
    __shared__ uint32_t s_box[4][4];   // per wave: umin, umax, vmin, vmax
    __shared__ uint32_t s_sum[4];
    // only chunks of supports up to 32 are cell-sorted and bounded; the
    // blocked kernels of the larger supports take the records in any order
    const uint32_t c_end = plane_cfirst[nplanes];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int p = 0;   // chunks come in increasing order: the plane only moves forward
    for (uint32_t c = blockIdx.x - small_blocks; c < c_end; c += gridDim.x - small_blocks) {
        const Chunk ch = chunks[c];
        if (ch.len <= kWaveSortMax) continue;   // the wave sort's chunks
        while (p + 1 < nplanes && c >= plane_cfirst[p + 1]) ++p;
        int pp;
        uint32_t tile;
        bucket_plane_tile(planes[p], ch.bucket, &pp, &tile);
        const PlaneLayout pl = planes[pp];
        if (pl.cls >= 3) continue;
        const uint32_t tu0 = (tile % (uint32_t)pl.ntu) << pl.log2T;
        const uint32_t tv0 = (tile / (uint32_t)pl.ntu) << pl.log2T;
        const int ncell = pl.T * pl.T;
        for (int i = threadIdx.x; i < ncell; i += blockDim.x) hist[i] = 0;
        __syncthreads();
        uint32_t umin = 0xffu, umax = 0u, vmin = 0xffu, vmax = 0u;
        for (uint32_t i = threadIdx.x; i < ch.len; i += blockDim.x) {
            RecMeta m = smeta[ch.start + i];
            m_in[i] = m;
            p_in[i] = sperm[ch.start + i];
            uint32_t du = meta_ku(m) - tu0, dv = meta_kv(m) - tv0;
            atomicAdd(&hist[cell_key(du, dv, pl.log2T)], 1u);
            umin = min(umin, du);
            umax = max(umax, du);
            vmin = min(vmin, dv);
            vmax = max(vmax, dv);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            umin = min(umin, (uint32_t)__shfl_xor((int)umin, off, 64));
            umax = max(umax, (uint32_t)__shfl_xor((int)umax, off, 64));
            vmin = min(vmin, (uint32_t)__shfl_xor((int)vmin, off, 64));
            vmax = max(vmax, (uint32_t)__shfl_xor((int)vmax, off, 64));
        }
        if (lane == 0) {
            s_box[wave][0] = umin;
            s_box[wave][1] = umax;
            s_box[wave][2] = vmin;
            s_box[wave][3] = vmax;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < 4; ++w) {
                umin = min(umin, s_box[w][0]);
                umax = max(umax, s_box[w][1]);
                vmin = min(vmin, s_box[w][2]);
                vmax = max(vmax, s_box[w][3]);
            }
            chunks[c].bbox = umin | (umax << 8) | (vmin << 16) | (vmax << 24);
        }
        {
            // exclusive scan of the (up to 1024) cell counts: 4 per thread
            uint32_t loc[4], sum = 0;
            for (int k = 0; k < 4; ++k) {
                int i = threadIdx.x * 4 + k;
                loc[k] = (i < ncell) ? hist[i] : 0u;
                sum += loc[k];
            }
            uint32_t incl = sum;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t y = (uint32_t)__shfl_up((int)incl, d, 64);
                if (lane >= d) incl += y;
            }
            if (lane == 63) s_sum[wave] = incl;
            __syncthreads();
            uint32_t run = incl - sum;
            for (int w = 0; w < wave; ++w) run += s_sum[w];
            for (int k = 0; k < 4; ++k) {
                int i = threadIdx.x * 4 + k;
                if (i < ncell) hist[i] = run;
                run += loc[k];
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < ch.len; i += blockDim.x) {
            RecMeta m = m_in[i];
            uint32_t du = meta_ku(m) - tu0, dv = meta_kv(m) - tv0;
            uint32_t pos = atomicAdd(&hist[cell_key(du, dv, pl.log2T)], 1u);
            smeta[ch.start + pos] = m;
            sperm[ch.start + pos] = p_in[i];
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// compute_indices: the index rule written out per record (parity/debug)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void indices_kernel(DevGeom g, int64_t nrec,
                                                      const T *__restrict__ uvw,
                                                      int32_t *k_lo_u, int32_t *k_lo_v,
                                                      int32_t *o_u, int32_t *o_v, int32_t *plane,
                                                      uint8_t *valid, int64_t *d_nskipped) {
    __shared__ uint32_t s_skip;
    if (threadIdx.x == 0) s_skip = 0;
    __syncthreads();
    uint32_t skipped = 0;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nrec;
         r += (int64_t)gridDim.x * blockDim.x) {
        // k_lo and o are 0 for skipped records
        RecIndex ix = index_record<T>(g, uvw[3 * r], uvw[3 * r + 1], uvw[3 * r + 2]);
        k_lo_u[r] = ix.ku;
        k_lo_v[r] = ix.kv;
        o_u[r] = ix.ou;
        o_v[r] = ix.ov;
        plane[r] = ix.plane;
        valid[r] = (uint8_t)ix.valid;
        skipped += !ix.valid;
    }
    if (d_nskipped) {
        if (skipped) atomicAdd(&s_skip, skipped);
        __syncthreads();
        if (threadIdx.x == 0 && s_skip)
            atomicAdd((unsigned long long *)d_nskipped, (unsigned long long)s_skip);
    }
}

int grid_blocks(int64_t n, int threads) {
    int64_t b = (n + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > 8192) b = 8192;
    return (int)b;
}

}  // namespace

mg_status launch_compute_indices(const DevGeom &g, int64_t nrec, const void *uvw,
                                 mg_dtype uvw_dtype, int32_t *k_lo_u, int32_t *k_lo_v,
                                 int32_t *o_u, int32_t *o_v, int32_t *plane, uint8_t *valid,
                                 int64_t *d_nskipped, hipStream_t stream) {
    if (nrec == 0) return MG_OK;
    int nb = grid_blocks(nrec, 256);
    if (uvw_dtype == MG_F32)
        hipLaunchKernelGGL(indices_kernel<float>, dim3(nb), dim3(256), 0, stream, g, nrec,
                           (const float *)uvw, k_lo_u, k_lo_v, o_u, o_v, plane, valid, d_nskipped);
    else
        hipLaunchKernelGGL(indices_kernel<double>, dim3(nb), dim3(256), 0, stream, g, nrec,
                           (const double *)uvw, k_lo_u, k_lo_v, o_u, o_v, plane, valid,
                           d_nskipped);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("index kernel: ") + hipGetErrorString(e));
    return MG_OK;
}

namespace {
// index_taps_kernel and scatter_kernel for the call's types
template <typename T, typename TapT, bool LDS>
void launch_index(const PlanState &P, const void *taps, const void *uvw, int tap_blocks,
                  int tap_per_plane, int blocks, hipStream_t stream) {
    const size_t lds = LDS ? sizeof(uint32_t) * (size_t)P.nbuckets : 0;
    hipLaunchKernelGGL((index_taps_kernel<T, TapT, LDS>), dim3(tap_blocks + blocks), dim3(256),
                       lds, stream, P.geom, P.d_planes, P.nrec, (const T *)uvw, P.hist,
                       (int32_t)P.nbuckets, P.counters, tap_blocks, tap_per_plane,
                       (int32_t)(P.kind == MG_KERNEL_WPROJ), (const TapT *)taps, (TapT *)P.taps,
                       P.table_elems);
}

template <typename T, bool LDS>
void launch_index_t(const PlanState &P, const void *taps, const void *uvw, int tap_blocks,
                    int tap_per_plane, int blocks, hipStream_t stream) {
    switch (P.tap_dtype) {
    case MG_F16:
        launch_index<T, __half, LDS>(P, taps, uvw, tap_blocks, tap_per_plane, blocks, stream);
        break;
    case MG_BF16:
        launch_index<T, __hip_bfloat16, LDS>(P, taps, uvw, tap_blocks, tap_per_plane, blocks,
                                             stream);
        break;
    default:
        launch_index<T, float, LDS>(P, taps, uvw, tap_blocks, tap_per_plane, blocks, stream);
        break;
    }
}

template <typename T, bool LDS>
void launch_scatter(const PlanState &P, const void *uvw, int blocks, hipStream_t stream) {
    const size_t lds = LDS ? sizeof(uint32_t) * (size_t)P.nbuckets : 0;
    hipLaunchKernelGGL((scatter_kernel<T, LDS>), dim3(blocks), dim3(256), lds, stream, P.geom,
                       P.d_planes, P.nrec, (const T *)uvw, P.cursor, (int32_t)P.nbuckets,
                       P.counters, P.smeta, P.sperm);
}
}  // namespace

// A build is seven launches (six where one block scans the buckets, eight where
// the block sums are scanned, one more for more than kPlaneArgs planes, and the
// unit lists of supports above 32): the smallest calls are bound by the launches,
// about 6 us each.
mg_status plan_build(PlanState &P, const void *taps, const void *uvw, mg_dtype uvw_dtype,
                     hipStream_t stream) {
    const int64_t nrec = P.nrec;
    const int64_t nb = P.nbuckets;
    const uint32_t R = (uint32_t)P.R;
    const int np = P.nplanes_eff;
    const bool wproj = P.kind == MG_KERNEL_WPROJ;
    const int64_t nscan = (nb + kScanBlock - 1) / kScanBlock;

    // plane layouts and zeros, by kernels (no copies from the host, no memset
    // nodes, so the calls stay capturable)
    for (int p0 = 0; p0 < np; p0 += kPlaneArgs) {
        PlaneArgs a;
        const int n = std::min(kPlaneArgs, np - p0);
        std::copy(P.planes.begin() + p0, P.planes.begin() + p0 + n, a.pl);
        hipLaunchKernelGGL(setup_kernel, dim3(grid_blocks((nb + 3) / 4, 256)), dim3(256), 0,
                           stream, a, p0, n, P.d_planes, P.counters, P.group_nunits, np, P.hist,
                           nb);
    }
    int64_t most = 0;   // tap table entries of the largest plane
    for (const PlaneLayout &L : P.planes) {
        const int64_t w = (int64_t)P.geom.beta * L.S;
        most = std::max<int64_t>(most, wproj ? w * w : w);
    }
    const int tap_per_plane = (int)std::min<int64_t>(grid_blocks(most, 256), 1024);
    const int tap_blocks = tap_per_plane * np;
    const bool lds = nb <= kLdsBuckets && nrec <= kLdsCallRecords;
    const int blocks = lds ? (int)std::max<int64_t>(1, (nrec + kLdsRecords - 1) / kLdsRecords)
                           : grid_blocks(nrec, 256);
    const bool f32 = uvw_dtype == MG_F32;
    if (lds && f32)
        launch_index_t<float, true>(P, taps, uvw, tap_blocks, tap_per_plane, blocks, stream);
    else if (lds)
        launch_index_t<double, true>(P, taps, uvw, tap_blocks, tap_per_plane, blocks, stream);
    else if (f32)
        launch_index_t<float, false>(P, taps, uvw, tap_blocks, tap_per_plane, blocks, stream);
    else
        launch_index_t<double, false>(P, taps, uvw, tap_blocks, tap_per_plane, blocks, stream);
    const bool scanned = nscan > kScanSums;
    if (nscan > 1)
        hipLaunchKernelGGL(scan_reduce_kernel, dim3((unsigned)nscan), dim3(kScanThreads), 0,
                           stream, P.hist, nb, R, P.sums);
    if (scanned)
        hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kScanThreads), 0, stream, P.sums, nscan);
    hipLaunchKernelGGL(scan_chunks_kernel, dim3((unsigned)nscan), dim3(kScanThreads), 0, stream,
                       P.hist, nb, R, P.sums, (int32_t)scanned, P.cursor, P.bucket_cfirst, P.chunks, P.d_planes, np,
                       P.plane_cfirst, P.counters);
    if (nrec > 0) {
        if (lds && f32) launch_scatter<float, true>(P, uvw, blocks, stream);
        else if (lds) launch_scatter<double, true>(P, uvw, blocks, stream);
        else if (f32) launch_scatter<float, false>(P, uvw, blocks, stream);
        else launch_scatter<double, false>(P, uvw, blocks, stream);
    }
    // cell sort and bounding box of the chunks of the window gridders'
    // supports (up to 32): small chunks one per wave, the others one per
    // workgroup
    const int cus = device_cus();
    const int64_t chunks = std::min<int64_t>(P.max_chunks, nrec);   // at most
    const int small_blocks = (int)std::min<int64_t>(8 * cus, std::max<int64_t>(1, (chunks + 3) / 4));
    const int large_blocks = (int)std::min<int64_t>(
        resident_groups((const void *)chunk_sort_kernel, 256, 0),
        std::max<int64_t>(1, nrec / kWaveSortMax));
    hipLaunchKernelGGL(chunk_sort_kernel, dim3(small_blocks + large_blocks), dim3(256), 0, stream,
                       P.plane_cfirst, np, P.d_planes, P.chunks, P.smeta, P.sperm, small_blocks);
    // units of every plane group
    GroupList groups{};
    const int ngroups = plane_groups(P.planes, groups);
    // (a thread per tile and no stride loop: the wave's prefix sum takes every
    // tile once, so the launch has to cover them all, up to 65536 workgroups)
    int64_t tiles = 1;
    for (const PlaneLayout &L : P.planes) tiles = std::max(tiles, (int64_t)L.ntu * L.ntv);
    auto unit_lists = [&](const GroupList &list, int n) {
        if (n > 0)
            hipLaunchKernelGGL(unit_list_kernel, dim3((unsigned)((tiles + 255) / 256), n),
                               dim3(256), 0, stream, P.d_planes, list, P.bucket_cfirst, P.chunks, R,
                               P.units, P.group_nunits);
    };
    // Waves reserve their units as they come, which is nearly tile order where a
    // group has the launch to itself, and the last tiles, at the edge of the grid,
    // have the smallest units.  The blocked kernels of the largest supports have few
    // and long units and wait for the last one: their groups get a launch each,
    // except in calls small enough to be bound by launches.  W-projection benchmark
    // workload, S > 32: degridding 1.94 ms, between 1.97 and 2.35 with the groups
    // in one launch; gridding 1.39, 1.43 to 1.53.
    if (nrec > kLdsCallRecords) {
        GroupList rest{};
        int n = 0;
        for (int i = 0; i < ngroups; ++i) {
            GroupList own{};
            own.first[0] = groups.first[i];
            if (P.planes[groups.first[i]].cls == 3)
                unit_lists(own, 1);
            else
                rest.first[n++] = groups.first[i];
        }
        unit_lists(rest, n);
    } else {
        unit_lists(groups, ngroups);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("plan kernels: ") + hipGetErrorString(e));
    return MG_OK;
}

// Arena layout of a plan: every array starts on a kArenaAlign boundary.
namespace {
template <typename F>
size_t walk_arena(const PlanState &P, F &&place) {
    const int np = P.nplanes_eff;
    const int64_t nb = P.nbuckets;
    const int64_t nscan = (nb + kScanBlock - 1) / kScanBlock;
    const size_t n = (size_t)(P.nrec + kRecPad);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += arena_round(bytes);
        return at;
    };
    place(0, take(sizeof(PlaneLayout) * (size_t)np));
    place(1, take(P.taps_bytes));
    place(2, take(sizeof(RecMeta) * n));
    place(3, take(sizeof(uint32_t) * n));
    place(4, take(sizeof(Chunk) * (size_t)P.max_chunks));
    place(5, take(sizeof(uint32_t) * (size_t)(np + 1)));
    place(6, take(sizeof(uint32_t) * (size_t)(nb + 1)));
    place(7, take(sizeof(uint2) * (size_t)P.max_chunks));
    place(8, take(sizeof(uint32_t) * (size_t)np));
    place(9, take(sizeof(int64_t) * 6));
    place(10, take(sizeof(uint32_t) * (size_t)nb));
    place(12, take(sizeof(uint32_t) * (size_t)nb));
    place(13, take(sizeof(uint2) * (size_t)(nscan + 1)));
    return off;
}
}  // namespace

size_t plan_arena_bytes(const PlanState &P) {
    return walk_arena(P, [](int, size_t) {});
}

void plan_carve(PlanState &P, void *arena) {
    char *base = static_cast<char *>(arena);
    P.bytes = walk_arena(P, [&](int what, size_t at) {
        void *p = base + at;
        switch (what) {
        case 0: P.d_planes = static_cast<PlaneLayout *>(p); break;
        case 1: P.taps = p; break;
        case 2: P.smeta = static_cast<RecMeta *>(p); break;
        case 3: P.sperm = static_cast<uint32_t *>(p); break;
        case 4: P.chunks = static_cast<Chunk *>(p); break;
        case 5: P.plane_cfirst = static_cast<uint32_t *>(p); break;
        case 6: P.bucket_cfirst = static_cast<uint32_t *>(p); break;
        case 7: P.units = static_cast<uint2 *>(p); break;
        case 8: P.group_nunits = static_cast<uint32_t *>(p); break;
        case 9: P.counters = static_cast<int64_t *>(p); break;
        case 10: P.hist = static_cast<uint32_t *>(p); break;
        case 12: P.cursor = static_cast<uint32_t *>(p); break;
        default: P.sums = static_cast<uint2 *>(p); break;
        }
    });
}

}  // namespace mg
