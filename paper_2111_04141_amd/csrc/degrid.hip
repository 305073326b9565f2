// Degridding (gather): vis_out[r] = sum_{i,j} conj(w_ij) G[k_lo + (i, j)], the
// adjoint of the gridding map.
//
// Supports above 32 (degrid_block_kernel): work unit a unit, the chunks of
// one tile over the planes of the launch's group.  The grid region the unit
// can touch (its tile plus the group's largest S - 1 halo) is cut into
// 8 x 8-cell blocks, one cell per lane; block b belongs to wave b mod NW and
// its 4 polarisations stay in registers for the whole unit, so the grid is
// read once per unit with coalesced loads.  Every wave walks all records of
// the unit's chunks (scalar loads).  Per record, a vector compare and a ballot give the wave's blocks
// that the footprint overlaps; each takes one tap load and 16 multiply-adds
// per lane into the record's partial sums.  Partial sums of B records are
// then reduced across the wave's lanes (a butterfly that halves the values
// each lane holds at every step) and across the waves through LDS, and one
// thread per (record, component) writes the result.  Supports 17 to 32 take
// degrid_taps_kernel, up to 16 degrid_cells_kernel (below).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace mg {

namespace {

struct DegridParams {
    int32_t npol, nu, nv, beta;
    int32_t p_lo, p_hi;
    uint32_t conj_base;   // element offset of the conjugated copy of the bank
    uint32_t tab_bytes;   // cells kernel: LDS for a plane's tap table
};

// Next unit of this launch after a workgroup's first, its own number (one
// vector atomic per unit and workgroup).
__device__ inline uint32_t next_unit_dg(uint32_t *queue, uint32_t *slot) {
    __syncthreads();
    if (threadIdx.x == 0) *slot = gridDim.x + atomicAdd(queue, 1u);
    __syncthreads();
    return uniform_u32(*slot);
}

// Reduce-scatter over the 64 lanes of a wave.  On entry every lane holds N
// partial values (N a power of two, 2..32); on exit v[0] of lane l holds the
// wave-wide sum of value index reduce_index<N>(l).  Each halving step pairs
// every lane with the lane that differs in one bit: a lane keeps the half of
// its values selected by that bit and adds the partner's copy of the same
// half.  The bits are taken in the order 32, 16 (the gfx950 half-wave and
// row swaps, which exchange two registers in one instruction), then 8, 2, 1
// (DPP row rotation and quad permutes), then 4 (a swizzle); steps beyond
// log2(N) only add the partner's value, so lanes differing in those bits end
// with the same sum.
__device__ constexpr int kReduceBits[6] = {32, 16, 8, 2, 1, 4};

__device__ inline float dpp_xor(float x, int o) {
    const int xi = __float_as_int(x);
    int r;
    if (o == 8)
        r = __builtin_amdgcn_update_dpp(0, xi, 0x128, 0xf, 0xf, false);   // row_ror:8
    else if (o == 2)
        r = __builtin_amdgcn_update_dpp(0, xi, 0x4e, 0xf, 0xf, false);    // quad_perm 2,3,0,1
    else
        r = __builtin_amdgcn_update_dpp(0, xi, 0xb1, 0xf, 0xf, false);    // quad_perm 1,0,3,2
    return __int_as_float(r);
}

template <int N, int S, int H>
__device__ inline void reduce_step(float (&v)[N], int lane) {
    constexpr int o = kReduceBits[S];
#pragma unroll
    for (int i = 0; i < H; ++i) {
        if constexpr (o == 32 || o == 16) {
            const auto r = (o == 32)
                               ? __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]),
                                                                  __float_as_uint(v[i + H]), false, false)
                               : __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]),
                                                                  __float_as_uint(v[i + H]), false, false);
            v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        } else {
            const bool up = (lane & o) != 0;
            const float keep = up ? v[i + H] : v[i];
            const float send = up ? v[i] : v[i + H];
            v[i] = keep + dpp_xor(send, o);
        }
    }
    if constexpr (H > 1) reduce_step<N, S + 1, H / 2>(v, lane);
}

template <int N>
__device__ inline void wave_reduce_scatter(float (&v)[N], int lane) {
    static_assert(N >= 2 && N <= 32 && (N & (N - 1)) == 0, "N: power of two in [2, 32]");
    reduce_step<N, 0, N / 2>(v, lane);
    constexpr int kSteps = __builtin_ctz(N);
#pragma unroll
    for (int s = kSteps; s < 6; ++s) {
        const int o = kReduceBits[s];
        v[0] += (o == 4 || o == 32 || o == 16) ? __shfl_xor(v[0], o) : dpp_xor(v[0], o);
    }
}

// Value index held by `lane` after wave_reduce_scatter<N>.
template <int N>
__device__ inline int reduce_index(int lane) {
    constexpr int kSteps = __builtin_ctz(N);
    int idx = 0;
#pragma unroll
    for (int s = 0; s < kSteps; ++s) idx = 2 * idx + ((lane & kReduceBits[s]) ? 1 : 0);
    return idx;
}

// One lane per value index writes it: the lanes whose non-halving bits are 0.
template <int N>
__device__ inline bool reduce_writer(int lane) {
    constexpr int kSteps = __builtin_ctz(N);
    int mask = 0;
#pragma unroll
    for (int s = kSteps; s < 6; ++s) mask |= kReduceBits[s];
    return (lane & mask) == 0;
}

template <int KMAX, int NW, int B, bool SEP, typename TapT>
__global__ __launch_bounds__(NW * kWave) void degrid_block_kernel(
    const RecMeta *__restrict__ smeta, const uint32_t *__restrict__ sperm,
    const float *__restrict__ grid, float *__restrict__ vis_out, const TapT *__restrict__ taps,
    const Chunk *__restrict__ chunks, const uint32_t *__restrict__ bucket_cfirst,
    const uint2 *__restrict__ units, const uint32_t *__restrict__ group_nunits,
    const PlaneLayout *__restrict__ planes, uint32_t *__restrict__ queue, DegridParams prm) {
    constexpr int NV = B * 8;   // partial values per lane: B records x 4 pol x (re, im)
    constexpr uint32_t kElem = SEP ? sizeof(TapT) : 2 * sizeof(TapT);
    __shared__ float s_part[2][NW][NV];
    __shared__ uint32_t s_next;
    const int wave = (int)uniform_u32(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int lu = lane & 7, lv = lane >> 3;
    const int npol = prm.npol;
    const char *tbase = reinterpret_cast<const char *>(taps);
    const int my_idx = reduce_index<NV>(lane);
    const bool writer = reduce_writer<NV>(lane);
    int parity = 0;

    // The launch covers one plane group; its work items are units (chunks of
    // one tile over the group's planes), whose grid values are loaded once
    // over the tile plus the group's largest halo.
    const PlaneLayout g0 = planes[prm.p_lo];
    const int Tm = g0.T - 1;
    const uint32_t ntu = (uint32_t)g0.ntu;
    const uint32_t gn = (uint32_t)g0.grp_n;
    const uint32_t gbase = (uint32_t)g0.base;
    const uint32_t nunits = group_nunits[prm.p_lo];
    const uint2 *gunits = units + bucket_cfirst[gbase];
    const int nbx = (g0.T + g0.grp_smax - 1 + 7) >> 3;
    const int nblocks = nbx * nbx;
    // lane k < KMAX: origin of the wave's block k, for the overlap tests
    uint32_t blo_u = 0xffff0000u, blo_v = 0xffff0000u;   // never overlaps
    {
        const int b = lane * NW + wave;
        if (lane < KMAX && b < nblocks) {
            blo_u = (uint32_t)((b % nbx) << 3);
            blo_v = (uint32_t)((b / nbx) << 3);
        }
    }
    // this lane's cell of each block (packed u | v << 16, region-relative)
    uint32_t cuv[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const int b = k * NW + wave;
        cuv[k] = (uint32_t)(((b % nbx) << 3) + lu) | ((uint32_t)(((b / nbx) << 3) + lv) << 16);
    }

    for (uint32_t it = blockIdx.x; it < nunits; it = next_unit_dg(queue, &s_next)) {
        const uint2 un = gunits[it];
        const uint32_t c0 = un.x, c1 = un.x + un.y;
        const uint32_t t = (chunks[c0].bucket - gbase) / gn;
        const int cu0 = (int)((t % ntu) << g0.log2T);
        const int cv0 = (int)((t / ntu) << g0.log2T);
        // this lane's grid values of each block
        float g[KMAX][8];
        bool bad = false;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const int b = k * NW + wave;
            const int u = cu0 + (int)(cuv[k] & 0xffffu), v = cv0 + (int)(cuv[k] >> 16);
            const bool in_grid = b < nblocks && u < prm.nu && v < prm.nv;
#pragma unroll
            for (int pol = 0; pol < 4; ++pol) {
                float2 x = make_float2(0.0f, 0.0f);
                if (in_grid && pol < npol)
                    x = *reinterpret_cast<const float2 *>(
                        grid + 2 * (((int64_t)pol * prm.nv + v) * prm.nu + u));
                g[k][2 * pol] = x.x;
                g[k][2 * pol + 1] = x.y;
                bad = bad || !isfinite(x.x) || !isfinite(x.y);
            }
        }
        // a zero tap times a non-finite grid value is NaN: units whose region
        // holds one mask the taps outside each footprint instead
        const bool exact = __syncthreads_or(bad) != 0;

        for (uint32_t c = c0; c < c1; ++c) {
            const Chunk ch = chunks[c];
            const int S = planes[g0.grp_first + (int)((ch.bucket - gbase) % gn)].S;
            // this lane's tap offset in each block, in bytes relative to the
            // footprint's first tap
            uint32_t voff[KMAX], voffv[KMAX];
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                const uint32_t cu = cuv[k] & 0xffffu, cv = cuv[k] >> 16;
                if constexpr (SEP) {
                    voff[k] = cu * kElem;
                    voffv[k] = cv * kElem;
                } else {
                    voff[k] = (cv * (uint32_t)S + cu) * kElem;
                    voffv[k] = 0u;
                }
            }

            auto visit = [&](const RecMeta m, float (&acc)[8], auto exact_t) {
                constexpr bool EXACT = decltype(exact_t)::value;
                const uint32_t a = meta_ku(m) & (uint32_t)Tm;
                const uint32_t bq = meta_kv(m) & (uint32_t)Tm;
                const uint32_t hit = (uint32_t)__ballot((blo_u + 7u - a <= (uint32_t)(S + 6)) &&
                                                        (blo_v + 7u - bq <= (uint32_t)(S + 6)));
                const uint32_t full = (uint32_t)__ballot((blo_u - a <= (uint32_t)(S - 8)) &&
                                                         (blo_v - bq <= (uint32_t)(S - 8)));
                const uint32_t ab = a | (bq << 16);
                const char *tb;
                const char *tbv = nullptr;
                if constexpr (SEP) {
                    tb = tbase + ((int64_t)(m.toff & 0xffffu) - (int64_t)a) * (int64_t)kElem;
                    tbv = tbase + ((int64_t)(m.toff >> 16) - (int64_t)bq) * (int64_t)kElem;
                } else {
                    tb = tbase +
                         ((int64_t)m.toff - (int64_t)(bq * (uint32_t)S + a)) * (int64_t)kElem;
                }
                auto tap = [&](const int k) {
                    uint32_t o = voff[k];
                    asm volatile("" : "+v"(o));   // keeps the offset 32-bit: scalar-base load
                    if constexpr (SEP) {
                        uint32_t ov = voffv[k];
                        asm volatile("" : "+v"(ov));
                        const float t = TapTraits<TapT>::real((const TapT *)(tb + o), 0) *
                                        TapTraits<TapT>::real((const TapT *)(tbv + ov), 0);
                        return make_float2(t, 0.0f);
                    } else {
                        return TapTraits<TapT>::cplx((const TapT *)(tb + o), 0);
                    }
                };
                // acc += conj(w) * G = (wr gr + wi gi) + j (wr gi - wi gr)
                auto madd = [&](const int k, const float2 w) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float gr = g[k][2 * q], gi = g[k][2 * q + 1];
                        acc[2 * q] = fmaf(w.x, gr, fmaf(w.y, gi, acc[2 * q]));
                        acc[2 * q + 1] = fmaf(w.x, gi, fmaf(-w.y, gr, acc[2 * q + 1]));
                    }
                };
                if constexpr (EXACT) {
#pragma unroll
                    for (int k = 0; k < KMAX; ++k) {
                        if (!((hit >> k) & 1u)) continue;
                        const uint32_t d = cuv[k] - ab;   // a borrow only where du < 0
                        if (((full >> k) & 1u) || max(d & 0xffffu, d >> 16) < (uint32_t)S)
                            madd(k, tap(k));
                    }
                } else {
                    float2 w[KMAX];
#pragma unroll
                    for (int k = 0; k < KMAX; ++k) {
                        w[k] = make_float2(0.0f, 0.0f);
                        if (!((hit >> k) & 1u)) continue;
                        const uint32_t d = cuv[k] - ab;
                        if (((full >> k) & 1u) || max(d & 0xffffu, d >> 16) < (uint32_t)S)
                            w[k] = tap(k);
                    }
#pragma unroll
                    for (int k = 0; k < KMAX; ++k)
                        if ((hit >> k) & 1u) madd(k, w[k]);
                }
            };

            auto records = [&](auto exact_t) {
                const uint32_t rend = ch.start + ch.len;
                // the next group's records are loaded while this group's taps are
                // (indices clamped into the chunk)
                RecMeta mnext[B];
                auto load_meta = [&](const uint32_t r) {
#pragma unroll
                    for (int bi = 0; bi < B; ++bi)
                        mnext[bi] = smeta[min(r + (uint32_t)bi, rend - 1)];
                };
                load_meta(ch.start);
                for (uint32_t r0 = ch.start; r0 < rend; r0 += B) {
                    const uint32_t nb = min((uint32_t)B, rend - r0);
                    // destination of the sums this thread writes (read now, used
                    // after the reductions)
                    const uint32_t dst = sperm[r0 + min((uint32_t)threadIdx.x >> 3, nb - 1)];
                    RecMeta m[B];
#pragma unroll
                    for (int bi = 0; bi < B; ++bi) m[bi] = mnext[bi];
                    load_meta(r0 + B);
                    float part[NV];
#pragma unroll
                    for (int i = 0; i < NV; ++i) part[i] = 0.0f;
#pragma unroll
                    for (int bi = 0; bi < B; ++bi) {
                        if ((uint32_t)bi < nb) {
                            float acc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                            visit(m[bi], acc, exact_t);
#pragma unroll
                            for (int q = 0; q < 8; ++q) part[bi * 8 + q] = acc[q];
                        }
                    }
                    wave_reduce_scatter<NV>(part, lane);
                    if (writer) s_part[parity][wave][my_idx] = part[0];
                    __syncthreads();
                    if ((int)threadIdx.x < NV) {
                        const int bi = threadIdx.x >> 3, q = threadIdx.x & 7;
                        if ((uint32_t)bi < nb && (q >> 1) < npol) {
                            float sum = 0.0f;
#pragma unroll
                            for (int w = 0; w < NW; ++w) sum += s_part[parity][w][threadIdx.x];
                            vis_out[((size_t)dst * npol + (q >> 1)) * 2 + (q & 1)] = sum;
                        }
                    }
                    // the other buffer takes the next group, so one barrier per
                    // group keeps the readers ahead of the next writers
                    parity ^= 1;
                }
            };
            if (exact)
                records(std::true_type{});
            else
                records(std::false_type{});
        }
    }
}

// Supports up to 16 (degrid_cells_kernel): a workgroup takes a unit (chunks of
// one tile over the planes of the group) and stages the unit's grid region once
// in LDS, 32 bytes a cell, [row][PITCH] cells of four float2 holding components
// (c, c + 4), c = 2 polarisation + part.
//
// Records come sorted by cell, so several share a footprint.  Where the plane's
// tap table is in LDS too, up to four records of one cell are taken together on
// the matrix cores: v_mfma_f32_4x4x1_16b multiplies four components of 16 cells
// (one cell per block, lane l holding component l % 4 of cell l / 4) by a tap of
// each of the four records (lane l: record l % 4), so a cell is read from LDS
// once for four records instead of once each; lane l ends with the components
// of record l % 4 over every 16th cell, and a reduction over 16 lanes finishes
// four records at once.  The real and imaginary taps sum apart (P = sum wr G,
// Q = sum wi G), and conj(w) G is put together at the end, with the sign of Q
// where the taps are the conjugated copy's.
// A record on its own costs about what it does in the lane-per-tap path (below)
// and four cost as much as one.  The lane-per-tap path reads 32 bytes of LDS a
// tap, 18 cycles for 64 taps shared by four SIMDs against 54 cycles of
// multiply-adds, and reduces every pair of records across the wave; it is kept
// for chunks too short to pay for the table, and tables that do not fit.
// Against the lane-per-tap path for all: 133.7M records of a W-projection bank,
// 8192^2, S <= 8 3.80 -> 2.84 ms, S <= 16 9.69 -> 7.74 ms (runs of 8 and 5 records
// a cell); separable 7 x 7, 10.08M records, 2048^2: 0.944 -> 0.522 ms.
// Sixteen waves to a workgroup: 9.3 ms for S <= 16.
//
// Lane-per-tap path: the lanes of a wave take the taps of one record (tap
// q = t * 64 + lane, q < S^2), so no lane sits outside a footprint; groups of B
// records are reduced across the wave's lanes.
constexpr int kCellWaves = 8;
constexpr int cells_smax(int ntap) { return ntap == 1 ? 8 : 16; }
constexpr int kCellTile = 16;
constexpr int cells_pitch(int ntap) { return kCellTile + cells_smax(ntap) - 1; }
// LDS of the region (bytes), before the tap table
constexpr size_t cells_region(int ntap) {
    return sizeof(float4) * 2 * (size_t)cells_pitch(ntap) * cells_pitch(ntap);
}
// LDS a workgroup's region and table may take so that two share a CU's 160 KB
constexpr size_t kCellLds = 80 * 1024 - 256;
// Records per oversampling phase a chunk needs for its plane's table to be
// copied to LDS (as the window gridders': the copy reads the table once; their
// figure, 8, is within 1 % on every timing case).
constexpr uint32_t kCellStagePerPhase = 16;
// Records per cell of its bounding box a chunk needs to be taken by cell: a
// group of one record costs half as much again as on the lane-per-tap path.
// 3.0M records of a bf16 bank, S <= 16, 2.6 records a cell: 264 us with two, 297
// without the rule.
constexpr uint32_t kDensePerCell = 2;

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int NTAP, int B, bool SEP, typename TapT>
__global__ __launch_bounds__(kWave * kCellWaves)
__attribute__((amdgpu_waves_per_eu(4))) void degrid_cells_kernel(
    const RecMeta *__restrict__ smeta, const uint32_t *__restrict__ sperm,
    const float *__restrict__ grid, float *__restrict__ vis_out, const TapT *__restrict__ taps,
    const Chunk *__restrict__ chunks, const uint32_t *__restrict__ bucket_cfirst,
    const uint2 *__restrict__ units, const uint32_t *__restrict__ group_nunits,
    const PlaneLayout *__restrict__ planes, uint32_t *__restrict__ queue, DegridParams prm) {
    constexpr int NV = B * 8;
    constexpr int kThreads = kWave * kCellWaves;
    constexpr int PITCH = cells_pitch(NTAP);
    constexpr uint32_t kElem = SEP ? sizeof(TapT) : 2 * sizeof(TapT);
    constexpr uint32_t kElemLds = SEP ? sizeof(float) : kElem;
    constexpr int kSteps = NTAP * 4;   // 16 cells each
    extern __shared__ float4 cells[];  // [PITCH][PITCH][2], then the tap table
    char *const s_reg = reinterpret_cast<char *>(cells);
    char *const s_tab = s_reg + cells_region(NTAP);
    __shared__ uint32_t s_next;
    const int wave = (int)uniform_u32(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int npol = prm.npol;
    const uint32_t beta = (uint32_t)prm.beta;
    const char *tbase = reinterpret_cast<const char *>(taps);
    const PlaneLayout gl = planes[prm.p_lo];
    const uint2 *gunits = units + bucket_cfirst[gl.base];
    const uint32_t nunits = group_nunits[prm.p_lo];
    int staged = -1;   // plane whose tap table is in LDS

    for (uint32_t it = blockIdx.x; it < nunits; it = next_unit_dg(queue, &s_next)) {
        const uint2 un = gunits[it];
        const uint32_t c0 = un.x, c1 = un.x + un.y;
        // region: union of the chunks' k_lo ranges extended by their supports
        uint32_t umin = 0xffu, vmin = 0xffu, uend = 0u, vend = 0u;
        for (uint32_t c = c0; c < c1; ++c) {
            const Chunk ch = chunks[c];
            int pc;
            uint32_t tile_;
            bucket_plane_tile(gl, ch.bucket, &pc, &tile_);
            const uint32_t Sc = (uint32_t)planes[pc].S;
            umin = min(umin, ch.bbox & 0xffu);
            vmin = min(vmin, (ch.bbox >> 16) & 0xffu);
            uend = max(uend, ((ch.bbox >> 8) & 0xffu) + Sc);
            vend = max(vend, (ch.bbox >> 24) + Sc);
        }
        uint32_t tile;
        {
            int pc;
            bucket_plane_tile(gl, chunks[c0].bucket, &pc, &tile);
        }
        const int cu0 = (int)(((tile % (uint32_t)gl.ntu) << gl.log2T) + umin);
        const int cv0 = (int)(((tile / (uint32_t)gl.ntu) << gl.log2T) + vmin);
        const int RW = (int)(uend - umin);
        const int RH = (int)(vend - vmin);

        // stage the region (cells outside it are never read); cell
        // j = rv * RW + ru, a thread stepping j by the workgroup size and
        // (rv, ru) by a fixed step (no division per cell)
        {
            const int ncells = RH * RW;
            const int step_u = kThreads % RW, step_v = kThreads / RW;
            int ru = (int)threadIdx.x % RW, rv = (int)threadIdx.x / RW;
            const float2 *gp = reinterpret_cast<const float2 *>(grid) + (int64_t)cv0 * prm.nu + cu0;
            const int64_t plane = (int64_t)prm.nv * prm.nu;
            for (int j = threadIdx.x; j < ncells; j += kThreads) {
                float2 x[4];
#pragma unroll
                for (int pol = 0; pol < 4; ++pol)
                    x[pol] = pol < npol ? gp[pol * plane + (int64_t)rv * prm.nu + ru]
                                        : make_float2(0.0f, 0.0f);
                float4 *dst = cells + 2 * (rv * PITCH + ru);
                dst[0] = make_float4(x[0].x, x[2].x, x[0].y, x[2].y);
                dst[1] = make_float4(x[1].x, x[3].x, x[1].y, x[3].y);
                ru += step_u;
                rv += step_v;
                if (ru >= RW) {
                    ru -= RW;
                    ++rv;
                }
            }
        }
        __syncthreads();

        uint32_t turn = 0;   // the wave whose turn it is, over the unit's groups
        for (uint32_t c = c0; c < c1; ++c) {
            const Chunk ch = chunks[c];
            int pc;
            uint32_t tile_;
            bucket_plane_tile(gl, ch.bucket, &pc, &tile_);
            const int S = planes[pc].S;
            const uint32_t tap_off = planes[pc].tap_off;
            const uint32_t ntap = beta * beta * (uint32_t)(S * S);   // phase-major S x S blocks
            // dense enough to be taken by cell
            const uint32_t box = (((ch.bbox >> 8) & 0xffu) - (ch.bbox & 0xffu) + 1u) *
                                 ((ch.bbox >> 24) - ((ch.bbox >> 16) & 0xffu) + 1u);
            const bool dense = ch.len >= kDensePerCell * box;
            bool in_lds = staged == pc;
            if (!in_lds && dense &&
                (gl.grp_n == 1 || ch.len >= kCellStagePerPhase * beta * beta) &&
                ntap * kElemLds <= prm.tab_bytes) {
                __syncthreads();   // the previous table's readers are done
                stage_taps<SEP, TapT>(s_tab, taps, tap_off, (uint32_t)S, beta, kThreads);
                __syncthreads();
                staged = pc;
                in_lds = true;
            }

            // up to four records of one cell at a time
            auto by_cell = [&]() {
                const int blk = lane >> 2, col = lane & 3;
                const int nsteps = (S * S + 15) >> 4;
                // this lane's cell of each step, as a byte offset from the
                // footprint's first cell (component pair `col`); cells past the
                // footprint read its first cell and count as zero
                uint32_t goff[kSteps];
#pragma unroll
                for (int t = 0; t < kSteps; ++t) {
                    const int q = t * 16 + blk;
                    const int qq = q < S * S ? q : 0;
                    const int j = qq / S;
                    goff[t] = (uint32_t)((j * PITCH + (qq - j * S)) * 32 + col * 8);
                }
                const bool rest = (S * S) % 16 != 0;
                const bool last_on = (nsteps - 1) * 16 + blk < S * S;
                const int idx = reduce_index<8>(lane);
                const uint32_t rb = ch.start + (uint32_t)(((uint64_t)ch.len * wave) / kCellWaves);
                const uint32_t re = ch.start + (uint32_t)(((uint64_t)ch.len * (wave + 1)) / kCellWaves);
                for (uint32_t r0 = rb; r0 < re; r0 += 64) {
                    // 64 records, one per lane: LDS offsets of the footprint and
                    // of the taps (bit 0: conjugated copy), destination
                    const uint32_t n = min(64u, re - r0);
                    const uint32_t r = r0 + min((uint32_t)lane, n - 1);
                    const RecMeta m = smeta[r];
                    const uint32_t perm = sperm[r];
                    uint32_t ph;
                    bool conj = false;
                    if constexpr (SEP) {
                        ph = ((m.toff >> 16) * beta + (m.toff & 0xffffu)) * (uint32_t)S;
                    } else {
                        conj = m.toff >= prm.conj_base;
                        ph = m.toff - tap_off - (conj ? prm.conj_base : 0u);
                    }
                    const uint32_t tt = ph * kElemLds | (conj ? 1u : 0u);
                    const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(
                        -1, (int)m.kuv, 0x138, 0xf, 0xf, false);   // wave_shr:1
                    const uint64_t starts = __ballot(m.kuv != prev || lane == 0);
                    for (uint32_t pos = 0; pos < n;) {
                        const uint64_t later = starts & (~0ull << pos << 1);
                        const uint32_t end = later ? min((uint32_t)__builtin_ctzll(later), n) : n;
                        const uint32_t g = min(4u, end - pos);
                        const uint32_t kuv = __builtin_amdgcn_readlane(m.kuv, pos);
                        const uint32_t cell0 = (((kuv >> 16) - (uint32_t)cv0) * PITCH +
                                                ((kuv & 0xffffu) - (uint32_t)cu0)) * 32u;
                        // this lane's record (the last one where there are fewer)
                        const int from = (int)((pos + min((uint32_t)col, g - 1)) << 2);
                        const uint32_t tj = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)tt);
                        const uint32_t dst = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)perm);
                        const char *tp = s_tab + (tj & ~1u) + blk * kElemLds;
                        f32x4 p0 = {0, 0, 0, 0}, p1 = p0, q0 = p0, q1 = p0;
                        // (compared step by step: the masks of all steps, kept
                        // for the loop, would spill)
                        int ns = nsteps, nrest = rest ? nsteps - 1 : -1;
                        asm volatile("" : "+s"(ns), "+s"(nrest));
#pragma unroll
                        for (int t0 = 0; t0 < kSteps; t0 += 4) {
                            if (t0 >= ns) break;
                            float2 w[4], x[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const int t = t0 + u;
                                if (t >= ns) continue;
                                const char *at = tp + t * 16 * (int)kElemLds;
                                if constexpr (SEP)
                                    w[u] = make_float2(*reinterpret_cast<const float *>(at), 0.0f);
                                else
                                    w[u] = TapTraits<TapT>::cplx(reinterpret_cast<const TapT *>(at), 0);
                                x[u] = *reinterpret_cast<const float2 *>(s_reg + (goff[t] + cell0));
                            }
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const int t = t0 + u;
                                if (t >= ns) continue;
                                if (t == nrest && !last_on)
                                    w[u] = x[u] = make_float2(0.0f, 0.0f);
                                p0 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[u].x, w[u].x, p0, 0, 0, 0);
                                p1 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[u].y, w[u].x, p1, 0, 0, 0);
                                if constexpr (!SEP) {
                                    q0 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[u].x, w[u].y, q0, 0, 0, 0);
                                    q1 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[u].y, w[u].y, q1, 0, 0, 0);
                                }
                            }
                        }
                        // conj(w) G = (wr gr + wi gi) + j (wr gi - wi gr)
                        float v[8];
                        const float sg = (tj & 1u) ? -1.0f : 1.0f;
#pragma unroll
                        for (int k = 0; k < 4; k += 2) {
                            v[k] = SEP ? p0[k] : fmaf(sg, q0[k + 1], p0[k]);
                            v[k + 1] = SEP ? p0[k + 1] : fmaf(-sg, q0[k], p0[k + 1]);
                            v[k + 4] = SEP ? p1[k] : fmaf(sg, q1[k + 1], p1[k]);
                            v[k + 5] = SEP ? p1[k + 1] : fmaf(-sg, q1[k], p1[k + 1]);
                        }
                        // over the lanes of the record (bits 2 to 5)
                        reduce_step<8, 0, 4>(v, lane);
                        v[0] += __shfl_xor(v[0], 4);
                        if ((lane & 4) == 0 && (uint32_t)col < g && (idx >> 1) < npol)
                            vis_out[((size_t)dst * npol + (idx >> 1)) * 2 + (idx & 1)] = v[0];
                        pos += g;
                    }
                }
            };

            // one record's taps across the wave, NT per lane
            auto by_tap = [&](auto nt_t) {
                constexpr int NT = decltype(nt_t)::value;
                const int my_idx = reduce_index<NV>(lane);
                const bool writer = reduce_writer<NV>(lane);
                // this lane's taps q = t * 64 + lane: LDS offset and table byte
                // offset relative to the footprint's first cell and first tap.
                // Taps t < NT - 1 lie in every footprint; where S^2 is not a
                // multiple of 64, lanes past S^2 in the last tap read the first
                // tap and first cell (in bounds) and their products are zeroed.
                const bool last_full = (S * S) % 64 == 0;
                const bool last_on = ((NT - 1) * 64 + lane) < S * S;
                int lg[NT];
                uint32_t lt[NT], ltv[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int qq = (t * 64 + lane < S * S) ? t * 64 + lane : 0;
                    const int j = qq / S, i = qq - j * S;
                    lg[t] = 2 * (j * PITCH + i);
                    if constexpr (SEP) {
                        lt[t] = (uint32_t)i * kElem;
                        ltv[t] = (uint32_t)j * kElem;
                    } else {
                        lt[t] = (uint32_t)(j * S + i) * kElem;
                        ltv[t] = 0u;
                    }
                }
                // groups of B records, taken by the waves in turn (continuing
                // from the unit's previous chunk); a short last group repeats
                // the chunk's last record (its sums are not written)
                const uint32_t rend = ch.start + ch.len;
                const uint32_t ngroups = (ch.len + B - 1) / B;
                const uint32_t gfirst = ((uint32_t)wave + kCellWaves - turn) % kCellWaves;
                turn = (turn + ngroups) % kCellWaves;
                // the records of this wave's next group are loaded while the
                // current group's taps are (indices clamped into the chunk)
                RecMeta mnext[B];
                auto load_meta = [&](const uint32_t g) {
#pragma unroll
                    for (int bi = 0; bi < B; ++bi)
                        mnext[bi] = smeta[min(ch.start + g * B + (uint32_t)bi, rend - 1)];
                };
                load_meta(gfirst);
                for (uint32_t gi = gfirst; gi < ngroups; gi += kCellWaves) {
                    const uint32_t r0 = ch.start + gi * B;
                    const uint32_t nb = min((uint32_t)B, rend - r0);
                    // destination of this lane's sum (read now, used after the
                    // reduction)
                    const uint32_t dst = sperm[r0 + min((uint32_t)(my_idx >> 3), nb - 1)];
                    float part[NV];
#pragma unroll
                    for (int i = 0; i < NV; ++i) part[i] = 0.0f;
                    // every tap of the group's records loaded, then the
                    // multiply-adds
                    float2 w[B][NT];
                    float4 ga[B][NT], gb[B][NT];
#pragma unroll
                    for (int bi = 0; bi < B; ++bi) {
                        const RecMeta m = mnext[bi];
                        const int sg = 2 * (((int)meta_kv(m) - cv0) * PITCH + ((int)meta_ku(m) - cu0));
                        const char *tb, *tbv = nullptr;
                        if constexpr (SEP) {
                            tb = tbase + (size_t)(m.toff & 0xffffu) * kElem;
                            tbv = tbase + (size_t)(m.toff >> 16) * kElem;
                        } else {
                            tb = tbase + (size_t)m.toff * kElem;
                        }
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            uint32_t o = lt[t], ov = ltv[t];
                            asm volatile("" : "+v"(o));   // keeps the offset 32-bit: scalar-base load
                            if constexpr (SEP) {
                                asm volatile("" : "+v"(ov));
                                w[bi][t] = make_float2(
                                    TapTraits<TapT>::real((const TapT *)(tb + o), 0) *
                                        TapTraits<TapT>::real((const TapT *)(tbv + ov), 0),
                                    0.0f);
                            } else {
                                w[bi][t] = TapTraits<TapT>::cplx((const TapT *)(tb + o), 0);
                            }
                            ga[bi][t] = cells[sg + lg[t]];
                            gb[bi][t] = cells[sg + lg[t] + 1];
                        }
                    }
                    load_meta(gi + kCellWaves);
#pragma unroll
                    for (int bi = 0; bi < B; ++bi) {
                        // lanes past S^2 in the last tap contribute nothing
                        if (!last_full && !last_on) {
                            w[bi][NT - 1] = make_float2(0.0f, 0.0f);
                            ga[bi][NT - 1] = gb[bi][NT - 1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                        }
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            // record bi's sums += conj(w) G
                            const float4 a4 = ga[bi][t], b4 = gb[bi][t];
                            const float gr[4] = {a4.x, b4.x, a4.y, b4.y};
                            const float gim[4] = {a4.z, b4.z, a4.w, b4.w};
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                float &ar = part[bi * 8 + 2 * q];
                                float &ai = part[bi * 8 + 2 * q + 1];
                                if constexpr (SEP) {
                                    ar = fmaf(w[bi][t].x, gr[q], ar);
                                    ai = fmaf(w[bi][t].x, gim[q], ai);
                                } else {
                                    ar = fmaf(w[bi][t].x, gr[q], fmaf(w[bi][t].y, gim[q], ar));
                                    ai = fmaf(w[bi][t].x, gim[q], fmaf(-w[bi][t].y, gr[q], ai));
                                }
                            }
                        }
                    }
                    wave_reduce_scatter<NV>(part, lane);
                    if (writer) {
                        const int bi = my_idx >> 3, q = my_idx & 7;
                        if ((uint32_t)bi < nb && (q >> 1) < npol)
                            vis_out[((size_t)dst * npol + (q >> 1)) * 2 + (q & 1)] = part[0];
                    }
                }
            };
            if (in_lds && dense) {
                by_cell();
            } else {
                switch ((S * S + 63) >> 6) {
                case 1: by_tap(std::integral_constant<int, 1>{}); break;
                case 2: by_tap(std::integral_constant<int, (NTAP < 2 ? NTAP : 2)>{}); break;
                case 3: by_tap(std::integral_constant<int, (NTAP < 3 ? NTAP : 3)>{}); break;
                default: by_tap(std::integral_constant<int, NTAP>{}); break;
                }
            }
        }
    }
}

// Supports 17 to 32: the lanes of a wave take the taps of one record (tap
// q = t * 64 + lane, q < S^2), so no lane sits outside a footprint.  A
// workgroup takes a unit (chunks of one tile over the planes of the group);
// the unit's grid region is staged once in LDS as [row][pol][col] float2
// rows of PITCH columns (a row stride of 4 PITCH + 8 float2, 16 banks
// modulo 64, spreads the rows of a footprint over the LDS banks); the
// waves of the workgroup take groups of B records in turn, and each group's
// sums are reduced across the wave's lanes only.
template <int PITCH>
constexpr int row_stride() { return 4 * PITCH + 8; }

// Waves per workgroup of the taps kernel: eight share each staged region, whose
// LDS limits how many workgroups a CU holds.
constexpr int kTapWaves = 8;
// Records per reduction group: two, as a lane holds several taps (registers; the
// reduction costs about the same per record either way).
constexpr int kTapRecords = 2;

template <int NTAP, int PITCH, int B, bool SEP, typename TapT>
__global__ __launch_bounds__(kWave * kTapWaves) void degrid_taps_kernel(
    const RecMeta *__restrict__ smeta, const uint32_t *__restrict__ sperm,
    const float *__restrict__ grid, float *__restrict__ vis_out, const TapT *__restrict__ taps,
    const Chunk *__restrict__ chunks, const uint32_t *__restrict__ bucket_cfirst,
    const uint2 *__restrict__ units, const uint32_t *__restrict__ group_nunits,
    const PlaneLayout *__restrict__ planes, uint32_t *__restrict__ queue, DegridParams prm) {
    constexpr int NV = B * 8;
    constexpr int kWaves = kTapWaves;
    constexpr int kThreads = kWave * kWaves;
    constexpr uint32_t kElem = SEP ? sizeof(TapT) : 2 * sizeof(TapT);
    constexpr int kPitch = PITCH;
    constexpr int kRowStride = row_stride<PITCH>();
    extern __shared__ float2 region[];   // [row][pol][PITCH], row stride kRowStride
    __shared__ uint32_t s_next;
    const int wave = (int)uniform_u32(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int npol = prm.npol;
    const char *tbase = reinterpret_cast<const char *>(taps);
    const int my_idx = reduce_index<NV>(lane);
    const bool writer = reduce_writer<NV>(lane);
    // the launch covers one plane group; its work items are the group's
    // units (chunks of one tile over the group's planes), whose region is
    // staged once for all their chunks
    const PlaneLayout gl = planes[prm.p_lo];
    const uint2 *gunits = units + bucket_cfirst[gl.base];
    const uint32_t nunits = group_nunits[prm.p_lo];

    for (uint32_t it = blockIdx.x; it < nunits; it = next_unit_dg(queue, &s_next)) {
        const uint2 un = gunits[it];
        const uint32_t c0 = un.x, c1 = un.x + un.y;
        // region: union of the chunks' k_lo ranges extended by their supports
        uint32_t umin = 0xffu, vmin = 0xffu, uend = 0u, vend = 0u;
        for (uint32_t c = c0; c < c1; ++c) {
            const Chunk ch = chunks[c];
            int pc;
            uint32_t tile_;
            bucket_plane_tile(gl, ch.bucket, &pc, &tile_);
            const uint32_t Sc = (uint32_t)planes[pc].S;
            umin = min(umin, ch.bbox & 0xffu);
            vmin = min(vmin, (ch.bbox >> 16) & 0xffu);
            uend = max(uend, ((ch.bbox >> 8) & 0xffu) + Sc);
            vend = max(vend, (ch.bbox >> 24) + Sc);
        }
        uint32_t tile;
        {
            int pc;
            bucket_plane_tile(gl, chunks[c0].bucket, &pc, &tile);
        }
        const int cu0 = (int)(((tile % (uint32_t)gl.ntu) << gl.log2T) + umin);
        const int cv0 = (int)(((tile / (uint32_t)gl.ntu) << gl.log2T) + vmin);
        const int RW = (int)(uend - umin);
        const int RH = (int)(vend - vmin);

        // stage the region (cells outside it are never read); cell
        // j = rv * RW + ru of each polarisation, a thread stepping j by the
        // workgroup size and (rv, ru) by a fixed step (no division per cell)
        {
            const int cells = RH * RW;
            const int step_u = kThreads % RW, step_v = kThreads / RW;
            const int ru0 = (int)threadIdx.x % RW, rv0 = (int)threadIdx.x / RW;
            for (int pol = 0; pol < npol; ++pol) {
                const float2 *gp = reinterpret_cast<const float2 *>(grid) +
                                   ((int64_t)pol * prm.nv + cv0) * prm.nu + cu0;
                int ru = ru0, rv = rv0;
                for (int j = threadIdx.x; j < cells; j += kThreads) {
                    region[rv * kRowStride + pol * kPitch + ru] = gp[(int64_t)rv * prm.nu + ru];
                    ru += step_u;
                    rv += step_v;
                    if (ru >= RW) {
                        ru -= RW;
                        ++rv;
                    }
                }
            }
        }
        __syncthreads();

        uint32_t turn = 0;   // the wave whose turn it is, over the unit's groups
        for (uint32_t c = c0; c < c1; ++c) {
            const Chunk ch = chunks[c];
            int pc;
            uint32_t tile_;
            bucket_plane_tile(gl, ch.bucket, &pc, &tile_);
            const int S = planes[pc].S;

            // this lane's taps q = t * 64 + lane: LDS offset and table byte
            // offset relative to the footprint's first cell and first tap.
            // Taps t < nt - 1 lie in every footprint; where S^2 is not a
            // multiple of 64, lanes past S^2 in the last tap read the first
            // tap and first cell (in bounds) and their products are zeroed.
            const int nt_rt = (S * S + 63) >> 6;
            const bool last_full = (S * S) % 64 == 0;
            const bool last_on = ((nt_rt - 1) * 64 + lane) < S * S;
            // NTAP taps held per lane, the chunk's count tested
            auto run = [&]() {
                constexpr int NT = NTAP;
                const int nt = nt_rt;
                int lg[NT];
                uint32_t lt[NT], ltv[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int q = min(t * 64 + lane, S * S - 1);
                    const int qq = (t * 64 + lane < S * S) ? q : 0;
                    const int j = qq / S, i = qq - (qq / S) * S;
                    lg[t] = j * kRowStride + i;
                    if constexpr (SEP) {
                        lt[t] = (uint32_t)i * kElem;
                        ltv[t] = (uint32_t)j * kElem;
                    } else {
                        lt[t] = (uint32_t)(j * S + i) * kElem;
                        ltv[t] = 0u;
                    }
                }
                // the last tap's offsets (its index is a run-time value: picked
                // once per chunk)
                int lg_last = lg[0];
                uint32_t lt_last = lt[0], ltv_last = ltv[0];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (t == nt - 1) {
                        lg_last = lg[t];
                        lt_last = lt[t];
                        ltv_last = ltv[t];
                    }
                }

                // groups of B records, taken by the waves in turn (continuing
                // from the unit's previous chunk); a short last group repeats
                // the chunk's last record (its sums are not written)
                const uint32_t rend = ch.start + ch.len;
                const uint32_t ngroups = (ch.len + B - 1) / B;
                const uint32_t gfirst = ((uint32_t)wave + kWaves - turn) % kWaves;
                turn = (turn + ngroups) % kWaves;
                // the records of this wave's next group are loaded while the
                // current group's taps are (indices clamped into the chunk)
                RecMeta mnext[B];
                auto load_meta = [&](const uint32_t g) {
#pragma unroll
                    for (int bi = 0; bi < B; ++bi)
                        mnext[bi] = smeta[min(ch.start + g * B + (uint32_t)bi, rend - 1)];
                };
                load_meta(gfirst);
                for (uint32_t gi = gfirst; gi < ngroups; gi += kWaves) {
                    const uint32_t r0 = ch.start + gi * B;
                    const uint32_t nb = min((uint32_t)B, rend - r0);
                    // destination of this lane's sum (read now, used after the
                    // reduction)
                    const uint32_t dst = sperm[r0 + min((uint32_t)(my_idx >> 3), nb - 1)];
                    float part[NV];
#pragma unroll
                    for (int i = 0; i < NV; ++i) part[i] = 0.0f;
                    // record bi of the group: its LDS offset and tap pointers
                    int sg[B];
                    const char *tb[B];
                    const char *tbv[B];
#pragma unroll
                    for (int bi = 0; bi < B; ++bi) {
                        const RecMeta m = mnext[bi];
                        sg[bi] = ((int)meta_kv(m) - cv0) * kRowStride + ((int)meta_ku(m) - cu0);
                        if constexpr (SEP) {
                            tb[bi] = tbase + (size_t)(m.toff & 0xffffu) * kElem;
                            tbv[bi] = tbase + (size_t)(m.toff >> 16) * kElem;
                        } else {
                            tb[bi] = tbase + (size_t)m.toff * kElem;
                            tbv[bi] = nullptr;
                        }
                    }
                    load_meta(gi + kWaves);
                    // tap weight and the 4 grid values of one tap of record bi
                    auto load = [&](const int bi, const int g_off, uint32_t o, uint32_t ov,
                                    float2 &w, float2 (&gv)[4]) {
                        asm volatile("" : "+v"(o));   // keeps the offset 32-bit: scalar-base load
                        if constexpr (SEP) {
                            asm volatile("" : "+v"(ov));
                            w = make_float2(TapTraits<TapT>::real((const TapT *)(tb[bi] + o), 0) *
                                                TapTraits<TapT>::real((const TapT *)(tbv[bi] + ov), 0),
                                            0.0f);
                        } else {
                            w = TapTraits<TapT>::cplx((const TapT *)(tb[bi] + o), 0);
                        }
                        const float2 *gp = region + sg[bi] + g_off;
#pragma unroll
                        for (int q = 0; q < 4; ++q) gv[q] = gp[q * kPitch];
                    };
                    // lanes past S^2 in the last tap contribute nothing
                    auto mask_last = [&](float2 &w, float2 (&gv)[4]) {
                        if (!last_on) {
                            w = make_float2(0.0f, 0.0f);
#pragma unroll
                            for (int q = 0; q < 4; ++q) gv[q] = make_float2(0.0f, 0.0f);
                        }
                    };
                    // record bi's sums += conj(w) * G
                    auto fma4 = [&](const int bi, const float2 w, const float2 (&gv)[4]) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            float &ar = part[bi * 8 + 2 * q];
                            float &ai = part[bi * 8 + 2 * q + 1];
                            ar = fmaf(w.x, gv[q].x, fmaf(w.y, gv[q].y, ar));
                            ai = fmaf(w.x, gv[q].y, fmaf(-w.y, gv[q].x, ai));
                        }
                    };
#pragma unroll
                    for (int bi = 0; bi < B; ++bi) {
                        // many taps per lane: four at a time (their loads
                        // in flight together; the LDS region already
                        // limits the kernel to two waves per SIMD, so the
                        // registers are there)
#pragma unroll
                        for (int t = 0; t < NT - 1; t += 4) {
                            if (t < nt - 1) {
                                float2 w[4], gv[4][4];
#pragma unroll
                                for (int u = 0; u < 4; ++u)
                                    if (t + u < NT - 1 && t + u < nt - 1)
                                        load(bi, lg[t + u], lt[t + u], ltv[t + u], w[u], gv[u]);
#pragma unroll
                                for (int u = 0; u < 4; ++u)
                                    if (t + u < NT - 1 && t + u < nt - 1) fma4(bi, w[u], gv[u]);
                            }
                        }
                        float2 w, gv[4];
                        load(bi, lg_last, lt_last, ltv_last, w, gv);
                        if (!last_full) mask_last(w, gv);
                        fma4(bi, w, gv);
                    }
                    wave_reduce_scatter<NV>(part, lane);
                    if (writer) {
                        const int bi = my_idx >> 3, q = my_idx & 7;
                        if ((uint32_t)bi < nb && (q >> 1) < npol)
                            vis_out[((size_t)dst * npol + (q >> 1)) * 2 + (q & 1)] = part[0];
                    }
                }
            };
            run();
        }
    }
}

// Outputs of skipped records are zero: they follow the valid ones in the
// plan's sorted order.  Also clears the work counters.
__global__ __launch_bounds__(256) void zero_skipped_kernel(const int64_t *__restrict__ counters,
                                                           uint32_t *__restrict__ queues,
                                                           int32_t nplanes, int64_t nrec,
                                                           const uint32_t *__restrict__ sperm,
                                                           int32_t npol,
                                                           float2 *__restrict__ vis_out) {
    if (blockIdx.x == 0 && (int)threadIdx.x < nplanes) queues[threadIdx.x] = 0u;
    const int64_t nvalid = counters[1];
    for (int64_t i = nvalid + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nrec;
         i += (int64_t)gridDim.x * blockDim.x) {
        float2 *o = vis_out + (size_t)sperm[i] * npol;
        for (int q = 0; q < npol; ++q) o[q] = make_float2(0.0f, 0.0f);
    }
}

struct DegridPtrs {
    const RecMeta *smeta;
    const uint32_t *sperm;
    const float *grid;
    float *vis_out;
    const void *taps;
    const Chunk *chunks;
    const uint32_t *bucket_cfirst;
    const uint2 *units;
    const uint32_t *group_nunits;
    const PlaneLayout *planes;
    uint32_t *queue;
};

template <int KMAX, int NW, int B, bool SEP, typename TapT>
hipError_t launch_dg(const DegridPtrs &a, const DegridParams &prm, int tile, int smax,
                     hipStream_t stream) {
    // every block of the largest region has an owner
    const int side = (tile + smax - 1 + 7) / 8;
    if (side * side > KMAX * NW) return hipErrorInvalidValue;
    auto kern = degrid_block_kernel<KMAX, NW, B, SEP, TapT>;
    hipLaunchKernelGGL(kern, dim3(resident_groups((const void *)kern, NW * kWave, 0)),
                       dim3(NW * kWave), 0,
                       stream, a.smeta, a.sperm, a.grid, a.vis_out, (const TapT *)a.taps,
                       a.chunks, a.bucket_cfirst, a.units, a.group_nunits, a.planes, a.queue,
                       prm);
    return hipGetLastError();
}

template <int NTAP, int PITCH, bool SEP, typename TapT>
hipError_t launch_dt(const DegridPtrs &a, const DegridParams &prm, int tile, int smax,
                     hipStream_t stream) {
    // the region must fit the compile-time pitch and the taps the lanes
    if (tile + smax - 1 > PITCH || smax * smax > NTAP * 64) return hipErrorInvalidValue;
    const size_t lds = sizeof(float2) * (size_t)row_stride<PITCH>() * (size_t)(tile + smax - 1);
    auto kern = degrid_taps_kernel<NTAP, PITCH, kTapRecords, SEP, TapT>;
    constexpr int threads = kWave * kTapWaves;
    hipLaunchKernelGGL(kern, dim3(resident_groups((const void *)kern, threads, lds)),
                       dim3(threads), lds,
                       stream, a.smeta, a.sperm, a.grid, a.vis_out, (const TapT *)a.taps,
                       a.chunks, a.bucket_cfirst, a.units, a.group_nunits, a.planes, a.queue,
                       prm);
    return hipGetLastError();
}

// The cells kernel, with LDS for the largest tap table of the launch's planes
// that fits beside the region with two workgroups to a CU.
template <int NTAP, bool SEP, typename TapT>
hipError_t launch_dc(const DegridPtrs &a, DegridParams prm, int tile, int smax,
                     const PlaneLayout *planes, hipStream_t stream) {
    if (tile != kCellTile || smax > cells_smax(NTAP)) return hipErrorInvalidValue;
    size_t table = 0;
    for (int p = prm.p_lo; p < prm.p_hi; ++p) {
        const size_t w = (size_t)prm.beta * planes[p].S;
        const size_t t = w * w * (SEP ? sizeof(float) : 2 * sizeof(TapT));
        if (cells_region(NTAP) + t <= kCellLds) table = std::max(table, t);
    }
    table = (table + 7) & ~size_t(7);
    prm.tab_bytes = (uint32_t)table;
    // (16 cells past a table's end are read, and count as zero)
    const size_t lds = cells_region(NTAP) + table + (table ? 16 * 2 * sizeof(float) : 0);
    // records per reduction group of the lane-per-tap path: two where a lane
    // holds several taps (registers; the reduction costs about the same per
    // record either way)
    auto kern = degrid_cells_kernel<NTAP, (NTAP > 1 ? 2 : 4), SEP, TapT>;
    constexpr int threads = kWave * kCellWaves;
    hipLaunchKernelGGL(kern, dim3(resident_groups((const void *)kern, threads, lds)),
                       dim3(threads), lds, stream, a.smeta, a.sperm, a.grid, a.vis_out,
                       (const TapT *)a.taps, a.chunks, a.bucket_cfirst, a.units, a.group_nunits,
                       a.planes, a.queue, prm);
    return hipGetLastError();
}

template <bool SEP, typename TapT>
hipError_t launch_deg(int cls, const DegridPtrs &a, const DegridParams &prm, int tile, int smax,
                      const PlaneLayout *planes, hipStream_t stream) {
    switch (cls) {
    case 0: return launch_dc<1, SEP, TapT>(a, prm, tile, smax, planes, stream);
    case 1: return launch_dc<4, SEP, TapT>(a, prm, tile, smax, planes, stream);
    case 2: return launch_dt<16, 48, SEP, TapT>(a, prm, tile, smax, stream);
    default: return launch_dg<7, 16, 2, SEP, TapT>(a, prm, tile, smax, stream);
    }
}

template <bool SEP>
hipError_t launch_deg_t(mg_dtype dt, int cls, const DegridPtrs &a, const DegridParams &prm,
                        int tile, int smax, const PlaneLayout *planes, hipStream_t stream) {
    switch (dt) {
    case MG_F16: return launch_deg<SEP, __half>(cls, a, prm, tile, smax, planes, stream);
    case MG_BF16: return launch_deg<SEP, __hip_bfloat16>(cls, a, prm, tile, smax, planes, stream);
    default: return launch_deg<SEP, float>(cls, a, prm, tile, smax, planes, stream);
    }
}

}  // namespace

size_t degrid_scratch_bytes(const PlanState &P) {
    return arena_round(sizeof(uint32_t) * (size_t)P.nplanes_eff);
}

mg_status launch_degrid(const PlanState &P, const void *grid, void *vis_out, void *scratch,
                        hipStream_t stream) {
    if (P.nrec == 0) return MG_OK;
    const int np = P.nplanes_eff;
    uint32_t *queues = static_cast<uint32_t *>(scratch);
    hipError_t e = hipSuccess;
    if (!queues) {
        e = scratch_alloc((void **)&queues, degrid_scratch_bytes(P), stream);
        if (e != hipSuccess) return set_error(MG_ENOMEM, "degrid: work queue allocation failed");
    }
    {
        int64_t nb = (P.nrec + 255) / 256;
        if (nb > 4096) nb = 4096;
        hipLaunchKernelGGL(zero_skipped_kernel, dim3((unsigned)nb), dim3(256), 0, stream,
                           P.counters, queues, np, P.nrec, P.sperm, P.geom.npol,
                           (float2 *)vis_out);
    }
    DegridPtrs a{P.smeta,    P.sperm,         (const float *)grid, (float *)vis_out,
                 P.taps,     P.chunks,        P.bucket_cfirst,     P.units,
                 P.group_nunits, P.d_planes,  nullptr};
    DegridParams prm{P.geom.npol, P.geom.nu, P.geom.nv, P.geom.beta, 0, 0,
                     (uint32_t)P.geom.conj_base, 0};
    const bool sep = P.kind == MG_KERNEL_SEPARABLE;
    // one launch per run of consecutive planes of the same class
    int p0 = 0;
    while (p0 < np && e == hipSuccess) {
        int p1 = p0 + 1;
        int smax = P.planes[p0].S;
        while (p1 < np && P.planes[p1].cls == P.planes[p0].cls) {
            smax = std::max(smax, P.planes[p1].S);
            ++p1;
        }
        prm.p_lo = p0;
        prm.p_hi = p1;
        a.queue = queues + p0;
        const int cls = P.planes[p0].cls;
        e = sep ? launch_deg_t<true>(P.tap_dtype, cls, a, prm, P.planes[p0].T, smax,
                                     P.planes.data(), stream)
                : launch_deg_t<false>(P.tap_dtype, cls, a, prm, P.planes[p0].T, smax,
                                      P.planes.data(), stream);
        p0 = p1;
    }
    if (e == hipSuccess) e = hipGetLastError();
    if (!scratch) scratch_free(queues, stream);
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("degrid kernels: ") + hipGetErrorString(e));
    return MG_OK;
}

}  // namespace mg
