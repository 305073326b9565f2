// Gridding (scatter) kernels.
//
// Work unit: a run of chunks (up to R records each) of one uv tile over the
// planes of a group (consecutive planes of one support class), taken by one
// workgroup; units are handed out through a per-launch counter.
//
// Supports up to 32: moving window (grid_window_kernel).
//  * Each wave keeps a moving window of slots in registers: slot (su, sv)
//    owns the grid cells congruent to (su, sv) modulo S, so every record's
//    S x S footprint holds exactly one cell of each slot, and a slot's
//    accumulators (4 polarisations, complex) keep summing while its cell
//    stays inside the footprints of consecutive records.  This is the
//    owner-computes scheme of Romein's GPU gridder, which the thesis's
//    Convolutional Gridder builds on (Chapter 4); the slots are spread over
//    the 64 lanes of a wave (up to S = 16) or of a team of two waves (up to
//    S = 32), and the records come cell-sorted, so windows move rarely where
//    records are dense.
//  * When a slot's cell leaves the footprint its sums are committed into an
//    LDS copy of the unit's grid region (bounding box plus S-1 halo) shared
//    by the workgroup.  The region holds 32-bit fixed point: the gather
//    (gather_units_kernel) bounds every partial sum a unit can produce,
//    B = 2 * sum over its records of max|tap component of the record's
//    plane| * max|visibility component|, picks the power-of-two scale 2^e
//    that maps B to at most 2^30, and stores the unit's visibilities already
//    multiplied by 2^e (exact), so the accumulators hold fixed-point units
//    and a commit is one conversion, rounded to nearest, and one integer LDS
//    atomic per component (integer LDS atomics run at full wave rate, unlike
//    float LDS atomics, which serialise per lane).  The sums cannot overflow
//    and each commit is off by at most half a quantum 2^-e, which is below
//    2^-30 B (2^e is the largest power of two with 2^e B <= 2^30).  At the end
//    of the unit the region is converted back to FP32 (times 2^-e) and added
//    to the grid with float atomics, one per touched cell.
//
// Supports above 32: blocked output-stationary kernel (grid_block_kernel),
// for the sparse planes of large |w|; see the kernel's comment.
//
// All polarisations are handled per visit: one tap load feeds 4 complex
// multiply-adds (the thesis's Polarisation Gain, Section 3.5), on the matrix
// cores in the window kernel, on the vector units, with the records read on the
// scalar unit, in the block kernel and for supports 9 to 16 whose taps stay in
// global memory.  Each record carries the table offset of its first tap (in the
// conjugated copy of the bank for w < 0).
#include <hip/hip_runtime.h>

#include <algorithm>

#include <type_traits>

#include "internal.h"

namespace mg {

namespace {

constexpr uint32_t kNoCell = 0xffffffffu;
constexpr int kBatch = 2;   // records per batch of scalar loads
// the last batch of a range starts at most kBatch - 1 past its end and the
// read-ahead batch kBatch further: the sorted arrays are padded for that
static_assert(2 * kBatch - 1 <= kRecPad, "record read-ahead runs past the padding");

// Waits for every outstanding scalar load.  Called once after a record
// loop's first batch is issued: otherwise the compiler places the wait for
// that batch at the loop top, where (scalar loads complete out of order) it
// also waits for the next batch's loads on every iteration.
__device__ inline void wait_scalar_loads() { __builtin_amdgcn_s_waitcnt(0xC07F); }


// Nearest integer (halves round up) in one instruction: the fixed-point
// commit of an accumulator that is already in units of the quantum.
__device__ inline int32_t round_to_fixed(float x) {
    int32_t r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// Per-unit word written by the gather: bits 0-7 the fixed-point exponent e
// plus 128 (the unit's visibilities are stored times 2^e), bit 8 set if the
// unit commits in fixed point, bit 9 set if one of its visibilities is not
// finite.
constexpr int32_t kUnitFixed = 1 << 8;
constexpr int32_t kUnitNonFinite = 1 << 9;
__device__ inline int unit_scale(int32_t info) { return (info & 0xff) - 128; }

struct GridParams {
    int32_t npol, nu, nv, beta;
    int32_t p_lo, p_hi;       // planes handled by this launch
    uint32_t conj_base;       // element offset of the conjugated copy of the bank
    uint32_t tab_bytes;       // window kernels: LDS for a plane's tap table
};

// Two 16-bit lanes of a 32-bit word (packed 16-bit integer arithmetic).
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ inline u16x2 as_u16x2(uint32_t x) { return __builtin_bit_cast(u16x2, x); }
__device__ inline uint32_t as_u32(u16x2 x) { return __builtin_bit_cast(uint32_t, x); }
// a.u b.u + a.v b.v + c (modulo 2^32) in one instruction, for a and b holding
// (u, v) in their 16-bit halves
__device__ inline uint32_t dot_uv(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_udot2(as_u16x2(a), as_u16x2(b), c, false);
}

// Visibilities of one record, 4 polarisations.
struct RecVis {
    float vr[4], vi[4];
};

__device__ inline RecVis unpack_vis(const float4 v01, const float4 v23) {
    RecVis f;
    f.vr[0] = v01.x; f.vi[0] = v01.y; f.vr[1] = v01.z; f.vi[1] = v01.w;
    f.vr[2] = v23.x; f.vi[2] = v23.y; f.vr[3] = v23.z; f.vi[3] = v23.w;
    return f;
}

// acc += w * v for 4 polarisations: (wr + j wi)(vr + j vi) =
// wr vr - wi vi + j (wr vi + wi vr).  Records with w < 0 point into the
// conjugated copy of the bank, so no sign logic is needed here.
__device__ inline void fma_complex(float (&acc)[8], const float2 w, const RecVis &f) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc[2 * q] = fmaf(w.x, f.vr[q], fmaf(w.y, -f.vi[q], acc[2 * q]));
        acc[2 * q + 1] = fmaf(w.x, f.vi[q], fmaf(w.y, f.vr[q], acc[2 * q + 1]));
    }
}

__device__ inline void fma_real(float (&acc)[8], const float w, const RecVis &f) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc[2 * q] = fmaf(w, f.vr[q], acc[2 * q]);
        acc[2 * q + 1] = fmaf(w, f.vi[q], acc[2 * q + 1]);
    }
}

// Units are handed out through a per-launch counter (one vector atomic per
// unit and workgroup) after each workgroup's first, its own number, so
// workgroups that draw small units take more of them; unit sizes vary from one
// record to R.  Each workgroup sees its units in increasing order.
__device__ inline uint32_t next_unit(uint32_t *queue, uint32_t *slot) {
    __syncthreads();   // the previous value has been read by every wave
    if (threadIdx.x == 0) *slot = gridDim.x + atomicAdd(queue, 1u);
    __syncthreads();
    return uniform_u32(*slot);
}

// ---------------------------------------------------------------------------
// moving-window gridder (supports up to 32)
// ---------------------------------------------------------------------------
// A footprint's S^2 cells are held by slots, slot (su, sv) owning the cells
// congruent to it mod S.  TEAM waves share one footprint, each holding a
// contiguous share of q = ceil(S^2 / TEAM) slots, at most KMAX per lane
// (q <= 64 KMAX); the workgroup's NW / TEAM teams take consecutive parts of
// each chunk's records, each team with its own window.
// Each slot keeps its cell and the term cell_v S + cell_u (separable taps
// outside LDS: cell_u and cell_v) of its tap offset (bytes, modulo 2^32); a
// record adds its own term, so the slot's tap offset costs one addition per
// record, and only slots whose cell leaves the footprint do more work.
// Work items are units: chunks of one tile over the planes of the launch's
// group.  An item's sums go to an LDS region covering what its chunks can
// touch, in fixed point, and from there to the grid once per item.
//
// The multiply-adds run on the matrix cores: v_mfma_f32_4x4x1_16b takes four
// visibility components as its A column (broadcast to the 16 blocks) and one
// tap per lane as its B row, so lane l of the result holds four components of
// cell l, the layout the slots have anyway, and every product is one fused
// multiply-add, bit for bit what v_fma_f32 gives.  FP32 matrix and vector
// instructions do not overlap on a SIMD (measured: their times add), but the
// four matrix instructions of a complex tap take 43 cycles for 64 cells where
// sixteen v_fma_f32 take 54, and the visibilities need no scalar registers.
// The taps come from a copy of the plane's phase-major table in LDS where it
// fits (the launch's tab_bytes) and the chunk is long enough to pay for the
// copy: a load of 64 lanes of 4 or 8 bytes in a footprint's rotated order
// takes the CU's L1 17 cycles, shared by four SIMDs, and LDS 5.  A separable
// table is held as the S x S products of its phases, one load instead of two.
// Measured on 133.7M records of a W-projection bank, 8192^2, against scalar-unit
// visibilities, v_fma_f32 and global taps: S <= 8 3.28 -> 2.40 ms, S <= 16 6.99 ->
// 6.65 ms, S <= 32 6.57 -> 6.22 ms; separable 7 x 7, 10.08M records on 2048^2:
// 0.714 -> 0.426 ms.
// Supports 9 to 16 with their taps in global memory keep the vector units: their
// records are read on the scalar unit, in batches, by v_fma_f32 (the same bits),
// and where no chunk of the call can have its table in LDS four waves share a
// region, so that more regions fit a CU and a short chunk is cut into fewer
// parts.  Records spread evenly over 1024^2, matrix cores and eight waves in
// both: S = 16, W-projection, beta 8, 100,000 records of one polarisation 129 ->
// 91 us; 4M records: S = 12 909 -> 822, separable beta 64 715 -> 605.
// Waves per workgroup (NW): eight (two such workgroups share a CU's LDS for
// supports up to 32, and the instances with several slots per lane are held
// to four waves per SIMD: beyond 128 VGPRs the eight-slot instance ran a
// third slower at three waves per SIMD), or those four.
// Largest support of each window instance and its LDS region: 8 planes
// (polarisations x re/im) of int32, each plane kWindowTile + S - 1 cells
// square at most.  The plane stride is a compile-time constant, so the eight
// commits of a slot address one base with immediate offsets.
constexpr int kWindowTile = 16;
constexpr int window_smax(int kmax) { return kmax == 1 ? 8 : kmax == 4 ? 16 : 32; }
constexpr int window_plane(int kmax) {
    return (kWindowTile + window_smax(kmax) - 1) * (kWindowTile + window_smax(kmax) - 1);
}
// LDS words of a window instance before the tap table: the region and the
// unit slot, rounded to 8 bytes
constexpr int window_words(int kmax) { return 8 * window_plane(kmax) + 2; }
constexpr size_t window_lds(int kmax) { return sizeof(int32_t) * (size_t)window_words(kmax); }
// LDS a workgroup may take so that two share a CU's 160 KB
constexpr size_t kWindowLds = 80 * 1024;
// Records a chunk needs, per oversampling phase, for its plane's table to be
// copied to LDS: the copy reads the table once through an L1 of about 32 bytes
// a cycle, what the records would read themselves over 1 / kStagePerPhase of
// the chunk.  (16, the degridders' figure, is within 1 % on every timing case.)
constexpr uint32_t kStagePerPhase = 8;
// ... and in all: with chunks of fewer records (calls of less than half a million)
// four waves on global taps are the faster (100,000 records, W-projection, beta
// 2, S = 16, one polarisation: 128 -> 91 us).
constexpr uint32_t kStageLeast = 128;
__host__ __device__ constexpr uint32_t stage_records(uint32_t beta) {
    return kStagePerPhase * beta * beta > kStageLeast ? kStagePerPhase * beta * beta : kStageLeast;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// acc += a[0..3] b for every lane's b, a in lanes 4 BLOCK .. 4 BLOCK + 3
template <int BLOCK>
__device__ inline f32x4 mfma_col(float a, float b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, acc, 4, BLOCK, 0);
}

// the four complex sums of a slot += w times a record's visibilities
template <bool SEP>
__device__ inline void fma_record(f32x4 &a0, f32x4 &a1, const float2 w, const RecVis &f) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f32x4 &a = q < 2 ? a0 : a1;
        const int e = 2 * (q & 1);
        if constexpr (SEP) {
            a[e] = fmaf(w.x, f.vr[q], a[e]);
            a[e + 1] = fmaf(w.x, f.vi[q], a[e + 1]);
        } else {
            a[e] = fmaf(w.x, f.vr[q], fmaf(w.y, -f.vi[q], a[e]));
            a[e + 1] = fmaf(w.x, f.vi[q], fmaf(w.y, f.vr[q], a[e + 1]));
        }
    }
}

template <int KMAX, int TEAM, int NW, bool SEP, typename TapT>
__global__ __launch_bounds__(kWave * NW)
__attribute__((amdgpu_waves_per_eu(4))) void grid_window_kernel(
    const RecMeta *__restrict__ smeta, const float *__restrict__ svis, float *__restrict__ grid,
    const TapT *__restrict__ taps, const Chunk *__restrict__ chunks,
    const uint32_t *__restrict__ bucket_cfirst, const uint2 *__restrict__ units,
    const uint32_t *__restrict__ group_nunits, const PlaneLayout *__restrict__ planes,
    const int32_t *__restrict__ uinfo, uint32_t *__restrict__ queue, GridParams prm) {
    // (the eight-slot class has no room for a table beside its region)
    constexpr bool TABLE = KMAX < 8 && NW == 8;
    constexpr int NTEAMS = NW / TEAM;
    constexpr int PS = window_plane(KMAX);   // plane stride (cells)
    // [8][PS], plane q holding [RH][RW], then the workgroup's unit slot (the
    // region starts at LDS address 0, so commit addresses need no base), then
    // the tap table
    extern __shared__ int32_t region[];
    uint32_t *const s_next = reinterpret_cast<uint32_t *>(region + 8 * PS);
    char *const s_tab = reinterpret_cast<char *>(region + window_words(KMAX));
    constexpr uint32_t kElem = SEP ? sizeof(TapT) : 2 * sizeof(TapT);   // bytes per tap
    constexpr uint32_t kElemLds = SEP ? sizeof(float) : kElem;          // the same in LDS
    const int wave = (int)uniform_u32(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int team = wave / TEAM, member = wave % TEAM;
    const int npol = prm.npol;
    const char *tbase = reinterpret_cast<const char *>(taps);
    const uint32_t beta = (uint32_t)prm.beta;

    // sign of the second A column: (re, im) -> (-im, re)
    const uint32_t swap_sign = (lane & 1) ? 0u : 0x80000000u;
    const int rot16 = ((lane + 16) & 63) << 2;

    // the launch covers one plane group; its work items are the group's units
    const PlaneLayout gl = planes[prm.p_lo];
    const uint32_t ubase = bucket_cfirst[gl.base];
    const uint2 *gunits = units + ubase;
    const uint32_t nunits = group_nunits[prm.p_lo];
    int staged = -1;   // plane whose tap table is in LDS
    for (uint32_t it = blockIdx.x; it < nunits; it = next_unit(queue, s_next)) {
        const uint2 un = gunits[it];
        const uint32_t c0 = un.x, c1 = un.x + un.y;
        // the item's region: union of its chunks' k_lo ranges (relative to
        // the tile origin) extended by their supports
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
        const uint32_t cu0 = ((tile % (uint32_t)gl.ntu) << gl.log2T) + umin;
        const uint32_t cv0 = ((tile / (uint32_t)gl.ntu) << gl.log2T) + vmin;
        const int RW = (int)(uend - umin);
        // byte offset in a region plane of cell (u, v): 4 (u - cu0) + 4 RW (v - cv0),
        // as one dot product of the packed cell with (4, 4 RW) plus a constant
        const uint32_t rstep = 4u | ((uint32_t)(4 * RW) << 16);
        const uint32_t rbias = 0u - 4u * (cu0 + (uint32_t)RW * cv0);
        const int RH = (int)(vend - vmin);
        const int plane_cells = RH * RW;

        // the unit's fixed-point exponent (its visibilities come scaled by
        // 2^scale); units with a non-finite visibility, or whose bound
        // overflows FP32, commit straight to the grid in FP32 (scale 0)
        const int32_t info = (int32_t)uniform_u32((uint32_t)uinfo[ubase + it]);
        const bool use_lds = (info & kUnitFixed) != 0;
        const int scale = unit_scale(info);
        if (use_lds) {
            for (int q = 0; q < 8; ++q)
                for (int i = threadIdx.x; i < plane_cells; i += NW * kWave) region[q * PS + i] = 0;
            __syncthreads();
        }
        // adds a slot's sums to its cell (fixed point: rounded to the nearest
        // quantum)
        auto commit = [&](const f32x4 &s0, const f32x4 &s1, uint32_t cell_uv) {
            const uint32_t cu_ = cell_uv & 0xffffu, cv_ = cell_uv >> 16;
            if (use_lds) {
                // (the products are below 2^24 and the sum is the cell's
                // in-region offset, so the wrap of the bias cancels)
                int32_t *dst = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(region) +
                                                           dot_uv(cell_uv, rstep, rbias));
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    atomicAdd(&dst[q * PS], round_to_fixed(s0[q]));
                    atomicAdd(&dst[(q + 4) * PS], round_to_fixed(s1[q]));
                }
            } else {
#pragma unroll
                for (int pol = 0; pol < 4; ++pol) {
                    if (pol < npol) {
                        float *dst = grid + 2 * (((int64_t)pol * prm.nv + cv_) * prm.nu + cu_);
                        unsafeAtomicAdd(dst, pol < 2 ? s0[2 * pol] : s1[2 * pol - 4]);
                        unsafeAtomicAdd(dst + 1, pol < 2 ? s0[2 * pol + 1] : s1[2 * pol - 3]);
                    }
                }
            }
        };

        for (uint32_t c = c0; c < c1; ++c) {
            const Chunk ch = chunks[c];
            int pc;
            uint32_t tile_;
            bucket_plane_tile(gl, ch.bucket, &pc, &tile_);
            const int S = planes[pc].S;
            const uint32_t tap_off = planes[pc].tap_off;
            const uint32_t ntap = beta * beta * (uint32_t)(S * S);   // phase-major S x S blocks
            bool in_lds = staged == pc;
            if (TABLE && !in_lds && ch.len >= stage_records(beta) &&
                ntap * kElemLds <= prm.tab_bytes) {
                __syncthreads();   // the previous table's readers are done
                stage_taps<SEP, TapT>(s_tab, taps, tap_off, (uint32_t)S, beta, NW * kWave);
                __syncthreads();
                staged = pc;
                in_lds = true;
            }

            // this wave's slots: member * q + k * 64 + lane (q = ceil(S^2 / TEAM));
            // per-lane flags are bit fields (bit k = slot k).  The slot count
            // per lane, KD = ceil(q / 64), is a compile-time constant of each
            // instance of the chunk's loop.
            const int nslots = S * S;
            const int q_ = (nslots + TEAM - 1) / TEAM;
            auto run = [&](auto kd_t, auto lds_t) {
                constexpr int KD = decltype(kd_t)::value;
                constexpr bool LDS = decltype(lds_t)::value;
                constexpr bool SEP1D = SEP && !LDS;   // two 1-D taps multiplied per record
                constexpr uint32_t kE = LDS ? kElemLds : kElem;
                // offset terms per cell step (bytes; phase-major table)
                const uint32_t su_step = kE;
                const uint32_t sv_step = SEP1D ? kE : (uint32_t)S * kE;
                // the same steps packed (u, v) for the dot product with a cell
                const uint32_t uv_step = su_step | (sv_step << 16);
                uint32_t cell[KD], lo[KD], lov[KD], suv[KD];
                uint32_t valid_bits = 0;
                f32x4 acc0[KD], acc1[KD];
#pragma unroll
                for (int k = 0; k < KD; ++k) {
                    const int j = k * kWave + lane;
                    uint32_t sidx = (uint32_t)(member * q_ + j);
                    if (j < q_ && sidx < (uint32_t)nslots) valid_bits |= 1u << k;
                    // a spare lane mirrors a real slot: it follows the same
                    // cells and reads the same (in-bounds) taps, and its sums
                    // are never committed
                    else sidx %= (uint32_t)nslots;
                    // slot (su, sv) owns the cells congruent to it mod S
                    const uint32_t sv = sidx / (uint32_t)S;
                    suv[k] = (sidx - sv * (uint32_t)S) | (sv << 16);
                    cell[k] = kNoCell;
                    lo[k] = 0u;
                    lov[k] = 0u;
                    acc0[k] = acc1[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                }

                // window of the footprint at kuv: slots whose cell left it commit
                // and take the cell congruent to them inside the new footprint
                auto window_update = [&](const uint32_t kuv) {
                    const uint32_t ku = kuv & 0xffffu, kv = kuv >> 16;
                    const uint32_t kmu = ku % (uint32_t)S, kmv = kv % (uint32_t)S;
                    // (u, v) pairs in 16-bit halves: the footprint origin, its
                    // residues mod S and S itself
                    const u16x2 korg = as_u16x2(kuv), kres = as_u16x2(kmu | (kmv << 16)),
                                ss = as_u16x2((uint32_t)S | ((uint32_t)S << 16));
#pragma unroll
                    for (int k = 0; k < KD; ++k) {
                        // the slot's cell has left the footprint (a borrow
                        // only where du < 0); the test runs on the exec mask
                        const uint32_t d = cell[k] - kuv;
                        if (max(d & 0xffffu, d >> 16) >= (uint32_t)S) {
                            if (((valid_bits >> k) & 1u) && cell[k] != kNoCell)
                                commit(acc0[k], acc1[k], cell[k]);
                            acc0[k] = acc1[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                            // the cell congruent to the slot in the footprint:
                            // origin + (slot - origin mod S) mod S, per half; a
                            // negative difference wraps above 2^15, and adding S
                            // brings it back below S, so the smaller of the two
                            // is the residue
                            const u16x2 dd = as_u16x2(suv[k]) - kres;
                            const u16x2 cc = korg + __builtin_elementwise_min(dd, dd + ss);
                            cell[k] = as_u32(cc);
                            // cells < 2^16 and steps < 2^10: the products
                            // and their sum are exact
                            if constexpr (SEP1D) {
                                lo[k] = dot_uv(cell[k], su_step, 0u);
                                lov[k] = dot_uv(cell[k], sv_step << 16, 0u);
                            } else {
                                lo[k] = dot_uv(cell[k], uv_step, 0u);
                            }
                        }
                    }
                };

                // A record's tap offset, relative to a slot's term, modulo 2^32:
                // computed by one lane per record, read back as a scalar.
                //   LDS: bytes into the plane's table; the conjugated copy of
                //   the bank (w < 0) is the sign of the imaginary taps, carried
                //   by the column they multiply
                //   global, separable: bytes of the u table, of the v table in offv
                //   global, W-projection: bytes relative to the record's phase,
                //   the phase (an element of the bank's table) in offv
                auto tap_term = [&](const RecMeta m, uint32_t *offv) {
                    const uint32_t ku = meta_ku(m), kv = meta_kv(m);
                    if constexpr (SEP1D) {
                        *offv = ((m.toff >> 16) - kv) * kE;
                        return ((m.toff & 0xffffu) - ku) * kE;
                    } else {
                        *offv = m.toff;
                        uint32_t ph = 0u;
                        if constexpr (SEP)
                            ph = ((m.toff >> 16) * beta + (m.toff & 0xffffu)) * (uint32_t)S;
                        else if constexpr (LDS)
                            ph = m.toff - tap_off - (m.toff >= prm.conj_base ? prm.conj_base : 0u);
                        return (ph - kv * (uint32_t)S - ku) * kE;
                    }
                };
                // taps of every slot for the record whose term is (t, tv)
                auto issue = [&](const uint32_t t, const uint32_t tv, float2 (&w)[KD]) {
#pragma unroll
                    for (int k = 0; k < KD; ++k) {
                        if constexpr (LDS) {
                            const char *at = s_tab + (lo[k] + t);
                            if constexpr (SEP)
                                w[k] = make_float2(*reinterpret_cast<const float *>(at), 0.0f);
                            else
                                w[k] = TapTraits<TapT>::cplx(reinterpret_cast<const TapT *>(at), 0);
                        } else if constexpr (SEP) {
                            uint32_t ou = lo[k] + t, ov = lov[k] + tv;
                            asm volatile("" : "+v"(ou));   // keeps the offset 32-bit: scalar-base load
                            asm volatile("" : "+v"(ov));
                            w[k] = make_float2(TapTraits<TapT>::real((const TapT *)(tbase + ou), 0) *
                                                   TapTraits<TapT>::real((const TapT *)(tbase + ov), 0),
                                               0.0f);
                        } else {
                            const char *tb = tbase + (size_t)tv * kE;
                            uint32_t o = lo[k] + t;
                            asm volatile("" : "+v"(o));
                            w[k] = TapTraits<TapT>::cplx((const TapT *)(tb + o), 0);
                        }
                    }
                };
                // (wr + j wi)(vr + j vi) = wr (vr, vi) + wi (-vi, vr): the
                // record's columns are blocks 2 HALF and 2 HALF + 1 of a and as
                auto madd = [&](const float2 (&w)[KD], const float a, const float as, auto half_t) {
                    constexpr int B0 = 2 * decltype(half_t)::value;
                    if constexpr (!SEP) {
#pragma unroll
                        for (int k = 0; k < KD; ++k) {
                            acc0[k] = mfma_col<B0>(as, w[k].y, acc0[k]);
                            acc1[k] = mfma_col<B0 + 1>(as, w[k].y, acc1[k]);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < KD; ++k) {
                        acc0[k] = mfma_col<B0>(a, w[k].x, acc0[k]);
                        acc1[k] = mfma_col<B0 + 1>(a, w[k].x, acc1[k]);
                    }
                };

                const uint32_t len = ch.len;
                const uint32_t rb = ch.start + (uint32_t)(((uint64_t)len * team) / NTEAMS);
                const uint32_t re = ch.start + (uint32_t)(((uint64_t)len * (team + 1)) / NTEAMS);
                if constexpr (KMAX == 4 && !LDS) {
                    // records on the scalar unit, in batches: the next batch's
                    // loads are issued after the current batch has been consumed
                    // (scalar loads complete out of order: waiting for one is
                    // waiting for all), so they overlap its multiply-adds
                    if (rb < re) {
                        RecMeta nm[kBatch];
                        float4 na4[kBatch], nb4[kBatch];
                        // the record arrays are padded (kRecPad entries), so a
                        // batch may run past the chunk's end (not used)
                        const RecMeta *pm = smeta + rb;
                        const float4 *pv = reinterpret_cast<const float4 *>(svis) + 2 * (size_t)rb;
                        auto load_batch = [&]() {
#pragma unroll
                            for (int i = 0; i < kBatch; ++i) {
                                nm[i] = pm[i];
                                na4[i] = pv[2 * i];
                                nb4[i] = pv[2 * i + 1];
                            }
                            pm += kBatch;
                            pv += 2 * kBatch;
                        };
                        uint32_t last_kuv = kNoCell;
                        load_batch();
                        wait_scalar_loads();
                        for (uint32_t r = rb; r < re; r += kBatch) {
                            RecMeta mm[kBatch];
                            float4 va4[kBatch], vb4[kBatch];
#pragma unroll
                            for (int i = 0; i < kBatch; ++i) {
                                mm[i] = nm[i];
                                va4[i] = na4[i];
                                vb4[i] = nb4[i];
                            }
                            __builtin_amdgcn_sched_barrier(0);
                            load_batch();
#pragma unroll
                            for (int i = 0; i < kBatch; ++i) {
                                if (r + (uint32_t)i < re) {
                                    if (mm[i].kuv != last_kuv) {
                                        last_kuv = mm[i].kuv;
                                        window_update(last_kuv);
                                    }
                                    const RecVis f = unpack_vis(va4[i], vb4[i]);
                                    uint32_t tv;
                                    const uint32_t t = tap_term(mm[i], &tv);
                                    float2 w[KD];
                                    issue(t, tv, w);
#pragma unroll
                                    for (int k = 0; k < KD; ++k)
                                        fma_record<SEP>(acc0[k], acc1[k], w[k], f);
                                }
                            }
                        }
#pragma unroll
                        for (int k = 0; k < KD; ++k)
                            if (((valid_bits >> k) & 1u) && cell[k] != kNoCell)
                                commit(acc0[k], acc1[k], cell[k]);
                    }
                } else if (rb < re) {
                    // eight records at a time: lane 8 i + c of `a` holds
                    // component c of record i; lanes past the range repeat its
                    // end.  Records go in pairs: the pair's columns are in
                    // lanes 0-15, and the register turns by 16 lanes after each
                    // pair (the block of an A column is an immediate of the
                    // instruction).
                    uint32_t last_kuv = kNoCell;
                    auto load_vis = [&](uint32_t r) {
                        return svis[min((uint64_t)8 * r + lane, (uint64_t)8 * re - 1)];
                    };
                    // n records whose meta is in lanes l0 .. l0 + n - 1 of m
                    // (terms t, tv), moved where bit l0 + i of `moves` is set
                    auto eight = [&](const uint32_t n, const uint32_t l0, const uint32_t kuv,
                                     const uint32_t t, const uint32_t tv, const uint32_t moves,
                                     float a, float as) {
                        auto fetch = [&](uint32_t i, float2 (&w)[KD]) {
                            issue(__builtin_amdgcn_readlane(t, i),
                                  LDS ? 0u : __builtin_amdgcn_readlane(tv, i), w);
                        };
                        auto turn = [&]() {
                            a = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute(
                                rot16, (int)__float_as_uint(a)));
                            if constexpr (!SEP)
                                as = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute(
                                    rot16, (int)__float_as_uint(as)));
                        };
                        float2 w[KD];
                        auto step = [&](uint32_t i, auto half_t) {
                            if ((moves >> (l0 + i)) & 1u)
                                window_update(__builtin_amdgcn_readlane(kuv, l0 + i));
                            fetch(l0 + i, w);
                            madd(w, a, as, half_t);
                        };
                        for (uint32_t i = 0; i < n; i += 2) {
                            step(i, std::integral_constant<int, 0>{});
                            if (i + 1 < n) {
                                step(i + 1, std::integral_constant<int, 1>{});
                                turn();
                            }
                        }
                    };
                    // (-im, re) columns: neighbours swapped, the first negated
                    auto swapped = [&](float a, uint32_t sign) {
                        return __uint_as_float(sign ^ (uint32_t)__builtin_amdgcn_update_dpp(
                                                          0, (int)__float_as_uint(a), 0xb1, 0xf,
                                                          0xf, false));
                    };
                    // bit i: the cell of the record in lane i differs from the
                    // previous record's
                    auto cell_changes = [&](uint32_t kuv) {
                        const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(
                            (int)last_kuv, (int)kuv, 0x138, 0xf, 0xf, false);   // wave_shr:1
                        return (uint32_t)__ballot(kuv != prev);
                    };
                    if constexpr (LDS) {
                        // the next eight records are loaded while these are used
                        // (their loads count apart from the taps' LDS reads)
                        RecMeta mn;
                        float an;
                        uint32_t tn = 0;
                        auto load = [&](uint32_t r) {
                            mn = smeta[min(r + (uint32_t)(lane & 7), re - 1)];
                            an = load_vis(r);
                            if constexpr (!SEP)
                                tn = smeta[min(r + (uint32_t)(lane >> 3), re - 1)].toff;
                        };
                        load(rb);
                        for (uint32_t r = rb; r < re; r += 8) {
                            const RecMeta mg = mn;
                            const float a = an;
                            float as = 0.0f;
                            if constexpr (!SEP)
                                as = swapped(a, swap_sign ^
                                                    (tn >= prm.conj_base ? 0x80000000u : 0u));
                            const uint32_t n = min(8u, re - r);
                            uint32_t tv;
                            const uint32_t t = tap_term(mg, &tv);
                            const uint32_t moves = cell_changes(mg.kuv);
                            last_kuv = __builtin_amdgcn_readlane(mg.kuv, n - 1);
                            if (r + 8 < re) load(r + 8);
                            eight(n, 0, mg.kuv, t, tv, moves, a, as);
                        }
                    } else {
                        // loads return in order, so the taps would wait for any
                        // records loaded ahead of them: 32 records at once
                        for (uint32_t r = rb; r < re; r += 32) {
                            const RecMeta mg = smeta[min(r + (uint32_t)(lane & 31), re - 1)];
                            float av[4];
#pragma unroll
                            for (int g = 0; g < 4; ++g) av[g] = load_vis(r + 8 * g);
                            uint32_t tv;
                            const uint32_t t = tap_term(mg, &tv);
                            const uint32_t moves = cell_changes(mg.kuv);
                            const uint32_t n = min(32u, re - r);
                            last_kuv = __builtin_amdgcn_readlane(mg.kuv, n - 1);
                            for (uint32_t g = 0; g < n; g += 8) {
                                eight(min(8u, n - g), g, mg.kuv, t, tv, moves, av[0],
                                      SEP ? 0.0f : swapped(av[0], swap_sign));
                                av[0] = av[1];
                                av[1] = av[2];
                                av[2] = av[3];
                            }
                        }
                    }
#pragma unroll
                    for (int k = 0; k < KD; ++k)
                        if (((valid_bits >> k) & 1u) && cell[k] != kNoCell)
                            commit(acc0[k], acc1[k], cell[k]);
                }
            };
            const int kdyn = (q_ + kWave - 1) / kWave;
            auto run_kd = [&](auto lds_t) {
                if constexpr (KMAX == 1) {
                    run(std::integral_constant<int, 1>{}, lds_t);
                } else if constexpr (KMAX == 4) {
                    switch (kdyn) {
                    case 1: run(std::integral_constant<int, 1>{}, lds_t); break;
                    case 2: run(std::integral_constant<int, 2>{}, lds_t); break;
                    case 3: run(std::integral_constant<int, 3>{}, lds_t); break;
                    default: run(std::integral_constant<int, 4>{}, lds_t); break;
                    }
                } else {
                    static_assert(KMAX == 8, "slot counts 1..8");
                    switch (kdyn) {
                    case 1: run(std::integral_constant<int, 1>{}, lds_t); break;
                    case 2: run(std::integral_constant<int, 2>{}, lds_t); break;
                    case 3: run(std::integral_constant<int, 3>{}, lds_t); break;
                    case 4: run(std::integral_constant<int, 4>{}, lds_t); break;
                    case 5: run(std::integral_constant<int, 5>{}, lds_t); break;
                    case 6: run(std::integral_constant<int, 6>{}, lds_t); break;
                    case 7: run(std::integral_constant<int, 7>{}, lds_t); break;
                    default: run(std::integral_constant<int, 8>{}, lds_t); break;
                    }
                }
            };
            if constexpr (!TABLE)
                run_kd(std::false_type{});
            else if (in_lds)
                run_kd(std::true_type{});
            else
                run_kd(std::false_type{});
        }

        if (use_lds) {
            __syncthreads();
            // word k of a polarisation is part k & 1 of cell k >> 1 = rv * RW + ru:
            // consecutive lanes add to consecutive words of a grid row, so an
            // atomic instruction covers its cache lines whole (the two parts
            // apart took 67 us for 100,800 records on 1024^2, this 44); a thread steps
            // its cell by half the workgroup, so (rv, ru) advance by a fixed
            // step (no division per cell)
            constexpr int kCells = NW * kWave / 2;
            const int part = threadIdx.x & 1, j0 = (int)threadIdx.x >> 1;
            const int step_u = kCells % RW, step_v = kCells / RW;
            const int ru0 = j0 % RW, rv0 = j0 / RW;
            for (int pol = 0; pol < npol; ++pol) {
                const int32_t *qp = region + (2 * pol + part) * PS;
                float *gp = grid + 2 * (((int64_t)pol * prm.nv + cv0) * prm.nu + cu0) + part;
                int ru_ = ru0, rv_ = rv0;
                for (int j = j0; j < plane_cells; j += kCells) {
                    const int32_t qv = qp[j];
                    if (qv != 0)
                        unsafeAtomicAdd(gp + 2 * ((int64_t)rv_ * prm.nu + ru_),
                                        ldexpf((float)qv, -scale));
                    ru_ += step_u;
                    rv_ += step_v;
                    if (ru_ >= RW) {
                        ru_ -= RW;
                        ++rv_;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// blocked output-stationary gridder (large supports)
// ---------------------------------------------------------------------------
// The grid region a unit can touch (its tile plus the group's largest S - 1
// halo) is cut into 8 x 8-cell blocks, one cell per lane; block b belongs to
// wave b mod NW of the workgroup (its k-th block is b = k NW + wave), and its
// 8 accumulators per lane stay in registers for the whole unit.  Every wave
// walks all records of the unit (scalar loads).  Per record, lane k of a
// wave tests block k against the record's footprint, so one vector compare
// and a ballot give the wave's overlapped blocks (and those lying wholly
// inside the footprint, which need no per-lane mask); each overlapped block
// then takes one tap load and 16 multiply-adds per lane.  Nothing is
// committed until the unit ends; then each touched cell is added to the
// grid with float atomics.  Where records are sparse, as in the high-|w|
// planes of large support, this replaces the moving window's per-record
// slot commits; the lane utilisation is S^2 over the overlapped blocks'
// cells, about (S/(S+7))^2.
// W-projection instances are held to 128 VGPRs (four waves per SIMD), which
// they fit without spilling; separable ones need a few more registers.
template <int KMAX, int NW, bool SEP, typename TapT>
__global__ __launch_bounds__(NW * kWave) __attribute__((amdgpu_waves_per_eu(SEP ? 1 : 4)))
void grid_block_kernel(
    const RecMeta *__restrict__ smeta, const float4 *__restrict__ svis, float *__restrict__ grid,
    const TapT *__restrict__ taps, const Chunk *__restrict__ chunks,
    const uint32_t *__restrict__ bucket_cfirst, const uint2 *__restrict__ units,
    const uint32_t *__restrict__ group_nunits, const PlaneLayout *__restrict__ planes,
    const int32_t *__restrict__ uinfo, uint32_t *__restrict__ queue, GridParams prm) {
    // Lanes outside a footprint normally multiply a zero tap, which adds
    // nothing; a non-finite visibility would turn that into NaN, so units
    // holding one take the masked path instead.
    constexpr uint32_t kElem = SEP ? sizeof(TapT) : 2 * sizeof(TapT);   // bytes per tap
    const int wave = (int)uniform_u32(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int lu = lane & 7, lv = lane >> 3;
    const int npol = prm.npol;
    const char *tbase = reinterpret_cast<const char *>(taps);

    // The launch covers one plane group.  Its work comes in units: chunks of
    // one tile (in any of the group's planes), accumulated together in
    // registers and committed once per unit over the tile's region (the
    // tile plus the group's largest halo).
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
    // per block: this lane's cell (packed u | v << 16, region-relative)
    uint32_t cuv[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const int b = k * NW + wave;
        cuv[k] = (uint32_t)(((b % nbx) << 3) + lu) | ((uint32_t)(((b / nbx) << 3) + lv) << 16);
    }

    __shared__ uint32_t s_next;
    const uint32_t ubase = bucket_cfirst[gbase];
    // the exact or fast path is chosen per unit
    for (uint32_t i = blockIdx.x; i < nunits; i = next_unit(queue, &s_next)) {
        const bool exact_unit =
            (uniform_u32((uint32_t)uinfo[ubase + i]) & (uint32_t)kUnitNonFinite) != 0u;
        auto work = [&](auto exact_t) {
            const uint2 un = gunits[i];
            const uint32_t c0 = un.x, c1 = un.x + un.y;
            const uint32_t t = (chunks[c0].bucket - gbase) / gn;
            const int cu0 = (int)((t % ntu) << g0.log2T);
            const int cv0 = (int)((t / ntu) << g0.log2T);

            float acc[KMAX][8];
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
#pragma unroll
                for (int q = 0; q < 8; ++q) acc[k][q] = 0.0f;
            uint32_t touched = 0;

            for (uint32_t c = c0; c < c1; ++c) {
                const Chunk ch = chunks[c];
                const int p = g0.grp_first + (int)((ch.bucket - gbase) % gn);
                const PlaneLayout pl = planes[p];
                const int S = pl.S;
                // this lane's tap offset in each block, in bytes relative to
                // the footprint's first tap
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

                auto visit = [&](const RecMeta m, const RecVis &f, auto exact_t) {
                    constexpr bool EXACT = decltype(exact_t)::value;
                    // footprint origin relative to the region
                    const uint32_t a = meta_ku(m) & (uint32_t)Tm;
                    const uint32_t bq = meta_kv(m) & (uint32_t)Tm;
                    // block [lo, lo+7] overlaps [a, a+S-1] iff lo + 7 - a in
                    // [0, S+6]; it lies inside iff lo - a in [0, S-8]
                    const uint32_t hit = (uint32_t)__ballot((blo_u + 7u - a <= (uint32_t)(S + 6)) &&
                                                            (blo_v + 7u - bq <= (uint32_t)(S + 6)));
                    const uint32_t full = (uint32_t)__ballot((blo_u - a <= (uint32_t)(S - 8)) &&
                                                             (blo_v - bq <= (uint32_t)(S - 8)));
                    touched |= hit;
                    const uint32_t ab = a | (bq << 16);
                    const char *tb_;
                    const char *tbv = nullptr;
                    if constexpr (SEP) {
                        tb_ = tbase + ((int64_t)(m.toff & 0xffffu) - (int64_t)a) * (int64_t)kElem;
                        tbv = tbase + ((int64_t)(m.toff >> 16) - (int64_t)bq) * (int64_t)kElem;
                    } else {
                        tb_ = tbase + ((int64_t)m.toff - (int64_t)(bq * (uint32_t)S + a)) * (int64_t)kElem;
                    }
                    // tap of lane's cell in block k (uniform base + 32-bit lane offset)
                    auto tap = [&](const int k) {
                        uint32_t o = voff[k];
                        asm volatile("" : "+v"(o));   // keeps the offset 32-bit: scalar-base load
                        if constexpr (SEP) {
                            uint32_t ov = voffv[k];
                            asm volatile("" : "+v"(ov));
                            const float t_ = TapTraits<TapT>::real((const TapT *)(tb_ + o), 0) *
                                             TapTraits<TapT>::real((const TapT *)(tbv + ov), 0);
                            return make_float2(t_, 0.0f);
                        } else {
                            return TapTraits<TapT>::cplx((const TapT *)(tb_ + o), 0);
                        }
                    };
                    auto madd = [&](const int k, const float2 w) {
                        if constexpr (SEP)
                            fma_real(acc[k], w.x, f);
                        else
                            fma_complex(acc[k], w, f);
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
                        // all tap loads of the record first, then the
                        // multiply-adds; lanes outside the footprint keep a
                        // zero tap (one vector test per overlapped block)
                        float2 w[KMAX];
#pragma unroll
                        for (int k = 0; k < KMAX; ++k) {
                            w[k] = make_float2(0.0f, 0.0f);
                            if (!((hit >> k) & 1u)) continue;
                            const uint32_t d = cuv[k] - ab;
                            if (max(d & 0xffffu, d >> 16) < (uint32_t)S) w[k] = tap(k);
                        }
#pragma unroll
                        for (int k = 0; k < KMAX; ++k)
                            if ((hit >> k) & 1u) madd(k, w[k]);
                    }
                };

                auto records = [&](auto exact_t) {
                    const uint32_t rb = ch.start, re = ch.start + ch.len;
                    RecMeta nm[kBatch];
                    float4 na4[kBatch], nb4[kBatch];
                    // the record arrays are padded (kRecPad entries), so a
                    // batch may run past the chunk's end (those are not used)
                    const RecMeta *pm = smeta + rb;
                    const float4 *pv = svis + 2 * (size_t)rb;
                    auto load_batch = [&]() {
#pragma unroll
                        for (int i = 0; i < kBatch; ++i) {
                            nm[i] = pm[i];
                            na4[i] = pv[2 * i];
                            nb4[i] = pv[2 * i + 1];
                        }
                        pm += kBatch;
                        pv += 2 * kBatch;
                    };
                    load_batch();
                    wait_scalar_loads();
                    for (uint32_t r = rb; r < re; r += kBatch) {
                        RecMeta mm[kBatch];
                        float4 va4[kBatch], vb4[kBatch];
#pragma unroll
                        for (int i = 0; i < kBatch; ++i) {
                            mm[i] = nm[i];
                            va4[i] = na4[i];
                            vb4[i] = nb4[i];
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        load_batch();
#pragma unroll
                        for (int i = 0; i < kBatch; ++i)
                            if (r + (uint32_t)i < re) visit(mm[i], unpack_vis(va4[i], vb4[i]), exact_t);
                    }
                };
                records(exact_t);
            }

            // commit: one float atomic per touched word.  A block's words go out
            // as two instructions of four rows each, lane l adding part l & 1 of
            // cell l >> 1 (fetched from the lane that holds the cell), so an
            // instruction covers 64 consecutive bytes of each row.
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                if (!((touched >> k) & 1u)) continue;
                const int b = k * NW + wave;
                const int u = cu0 + ((b % nbx) << 3) + ((lane >> 1) & 7);
                const int v = cv0 + ((b / nbx) << 3) + (lane >> 4);
                const int from = (lane >> 1) << 2;   // byte index of lane l >> 1
#pragma unroll
                for (int pol = 0; pol < 4; ++pol) {
                    if (pol >= npol) continue;
                    const int re = (int)__float_as_uint(acc[k][2 * pol]);
                    const int im = (int)__float_as_uint(acc[k][2 * pol + 1]);
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int xr = __builtin_amdgcn_ds_bpermute(from + 128 * half, re);
                        const int xi = __builtin_amdgcn_ds_bpermute(from + 128 * half, im);
                        const float x = __uint_as_float((uint32_t)((lane & 1) ? xi : xr));
                        const int vh = v + 4 * half;
                        if (x != 0.0f && u < prm.nu && vh < prm.nv)
                            unsafeAtomicAdd(grid + 2 * (((int64_t)pol * prm.nv + vh) * prm.nu + u) +
                                                (lane & 1),
                                            x);
                    }
                }
            }
        };
        if (exact_unit)
            work(std::true_type{});
        else
            work(std::false_type{});
    }
}

// Gathers the visibilities of the plane groups' units (one group per
// blockIdx.y) into sorted order, padded to 4 polarisations, writes each unit's
// word (see kUnitFixed) and clears the group's work counter.  A workgroup takes a
// unit (at most kGatherThreads * kGatherPerThread records, contiguous in sorted
// order): every thread first loads the
// permutation entries of its records, then their visibilities (all loads in
// flight together), bounds the unit's partial sums, and for the window
// classes (fixed = 1) stores the visibilities multiplied by the unit's
// power-of-two scale.
constexpr int kGatherThreads = 256;
constexpr int kGatherPerThread = 8;   // R <= 2048 records per unit

__global__ __launch_bounds__(kGatherThreads) void gather_units_kernel(
    const PlaneLayout *__restrict__ planes, GroupList groups, int32_t sep,
    uint32_t *__restrict__ queues, const uint32_t *__restrict__ bucket_cfirst, const uint2 *__restrict__ units,
    const uint32_t *__restrict__ group_nunits, const Chunk *__restrict__ chunks,
    const uint32_t *__restrict__ sperm, const float2 *__restrict__ vis, int32_t npol,
    const double *__restrict__ factor, float4 *__restrict__ svis, int32_t *__restrict__ uinfo) {
    __shared__ float s_part[kGatherThreads / kWave];
    __shared__ int s_bad[kGatherThreads / kWave];
    const int g = groups.first[blockIdx.y];
    if (blockIdx.x == 0 && threadIdx.x == 0) queues[g] = 0u;
    const PlaneLayout gl = planes[g];
    const bool fixed = gl.cls <= 2;
    const uint32_t ubase = bucket_cfirst[gl.base];
    const uint32_t n = group_nunits[g];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t it = blockIdx.x; it < n; it += gridDim.x) {
        const uint2 un = units[ubase + it];
        const uint32_t c0 = un.x, c1 = un.x + un.y;
        const uint32_t rs = chunks[c0].start;
        const Chunk last = chunks[c1 - 1];
        const uint32_t re = last.start + last.len;
        uint32_t idx[kGatherPerThread];
#pragma unroll
        for (int k = 0; k < kGatherPerThread; ++k) {
            const uint32_t r = rs + threadIdx.x + (uint32_t)k * kGatherThreads;
            idx[k] = (r < re) ? sperm[r] : 0u;
        }
        float4 a[kGatherPerThread], b[kGatherPerThread];
#pragma unroll
        for (int k = 0; k < kGatherPerThread; ++k) {
            const uint32_t r = rs + threadIdx.x + (uint32_t)k * kGatherThreads;
            a[k] = b[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (r >= re) continue;
            const float2 *v = vis + (size_t)idx[k] * npol;
            if (npol == 4) {
                a[k] = reinterpret_cast<const float4 *>(v)[0];
                b[k] = reinterpret_cast<const float4 *>(v)[1];
            } else {
                float2 x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = (q < npol) ? v[q] : make_float2(0.0f, 0.0f);
                a[k] = make_float4(x[0].x, x[0].y, x[1].x, x[1].y);
                b[k] = make_float4(x[2].x, x[2].y, x[3].x, x[3].y);
            }
        }
        if (factor) {
            const double f = *factor;
            auto times = [&](float x) { return (float)((double)x * f); };
#pragma unroll
            for (int k = 0; k < kGatherPerThread; ++k) {
                a[k] = make_float4(times(a[k].x), times(a[k].y), times(a[k].z), times(a[k].w));
                b[k] = make_float4(times(b[k].x), times(b[k].y), times(b[k].z), times(b[k].w));
            }
        }
        // bound: sum over the records of the plane's largest weight component
        // times the record's largest visibility component (the chunk of a
        // record, hence its plane, only moves forward with r)
        float part = 0.0f;
        bool bad = false;
        uint32_t c = c0;
        uint32_t cend = chunks[c0].start + chunks[c0].len;
        float wmax = 0.0f;
        {
            int pc;
            uint32_t tile_;
            bucket_plane_tile(gl, chunks[c0].bucket, &pc, &tile_);
            const float t = planes[pc].tmax;
            wmax = sep ? t * t : t;
        }
#pragma unroll
        for (int k = 0; k < kGatherPerThread; ++k) {
            const uint32_t r = rs + threadIdx.x + (uint32_t)k * kGatherThreads;
            if (r >= re) continue;
            while (r >= cend) {
                ++c;
                const Chunk ch = chunks[c];
                cend = ch.start + ch.len;
                int pc;
                uint32_t tile_;
                bucket_plane_tile(gl, ch.bucket, &pc, &tile_);
                const float t = planes[pc].tmax;
                wmax = sep ? t * t : t;
            }
            const float m = fmaxf(fmaxf(fmaxf(fabsf(a[k].x), fabsf(a[k].y)), fmaxf(fabsf(a[k].z), fabsf(a[k].w))),
                                  fmaxf(fmaxf(fabsf(b[k].x), fabsf(b[k].y)), fmaxf(fabsf(b[k].z), fabsf(b[k].w))));
            part += wmax * m;
            bad = bad || !(isfinite(a[k].x) && isfinite(a[k].y) && isfinite(a[k].z) &&
                           isfinite(a[k].w) && isfinite(b[k].x) && isfinite(b[k].y) &&
                           isfinite(b[k].z) && isfinite(b[k].w));
        }
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
        const bool wbad = __any(bad);
        if (lane == 0) {
            s_part[wave] = part;
            s_bad[wave] = wbad ? 1 : 0;
        }
        __syncthreads();
        float bound = 0.0f;
        int anybad = 0;
        for (int w = 0; w < kGatherThreads / kWave; ++w) {
            bound += s_part[w];
            anybad |= s_bad[w];
        }
        __syncthreads();   // s_part is rewritten by the next unit
        // margin for the rounding of the sums above
        bound = 2.0f * bound * 1.0001f + 1e-30f;
        int scale = 0;
        int32_t info = anybad ? kUnitNonFinite : 0;
        if (fixed && !anybad && isfinite(bound)) {
            int e = 0;
            frexpf(bound, &e);   // bound < 2^e
            scale = max(-120, min(120, 30 - e));
            info |= kUnitFixed;
        }
        info |= (scale + 128) & 0xff;
        if (threadIdx.x == 0) uinfo[ubase + it] = info;
        const float fs = ldexpf(1.0f, scale);
#pragma unroll
        for (int k = 0; k < kGatherPerThread; ++k) {
            const uint32_t r = rs + threadIdx.x + (uint32_t)k * kGatherThreads;
            if (r >= re) continue;
            float4 x = a[k], y = b[k];
            if (scale != 0) {
                x.x *= fs; x.y *= fs; x.z *= fs; x.w *= fs;
                y.x *= fs; y.y *= fs; y.z *= fs; y.w *= fs;
            }
            svis[2 * (size_t)r] = x;
            svis[2 * (size_t)r + 1] = y;
        }
    }
}

struct GridPtrs {
    const RecMeta *smeta;
    const float4 *svis;
    float *grid;
    const void *taps;
    const Chunk *chunks;
    const uint32_t *bucket_cfirst;
    const uint2 *units;
    const uint32_t *group_nunits;
    const PlaneLayout *planes;
    const int32_t *uinfo;        // per-unit words written by the gather
    uint32_t *queue;             // this launch's unit counter
};

// `table`: bytes of the largest tap table of the launch's planes that fits
// beside the region with two workgroups to a CU and that a chunk of the call can
// be long enough for (0: none).
template <int KMAX, int TEAM, int NW, bool SEP, typename TapT>
void launch_window(const GridPtrs &a, GridParams prm, size_t table, hipStream_t stream) {
    auto kern = grid_window_kernel<KMAX, TEAM, NW, SEP, TapT>;
    const int threads = kWave * NW;
    prm.tab_bytes = (uint32_t)table;
    const size_t lds = window_lds(KMAX) + table;
    hipLaunchKernelGGL(kern, dim3(resident_groups((const void *)kern, threads, lds)),
                       dim3(threads), lds, stream, a.smeta, (const float *)a.svis, a.grid, (const TapT *)a.taps,
                       a.chunks, a.bucket_cfirst, a.units, a.group_nunits, a.planes, a.uinfo,
                       a.queue, prm);
}

template <int KMAX, int NW, bool SEP, typename TapT>
void launch_block(const GridPtrs &a, const GridParams &prm, hipStream_t stream) {
    auto kern = grid_block_kernel<KMAX, NW, SEP, TapT>;
    hipLaunchKernelGGL(kern, dim3(resident_groups((const void *)kern, NW * kWave, 0)),
                       dim3(NW * kWave), 0, stream, a.smeta, a.svis, a.grid, (const TapT *)a.taps,
                       a.chunks, a.bucket_cfirst, a.units, a.group_nunits, a.planes, a.uinfo,
                       a.queue, prm);
}

// Largest region, in 8 x 8 blocks, of a chunk of tile side T and support S.
inline int region_blocks(int T, int S) {
    const int side = (T + S - 1 + 7) / 8;
    return side * side;
}

template <bool SEP, typename TapT>
hipError_t launch_class(int cls, const GridPtrs &a, const GridParams &prm, int smax, int tile,
                        const PlaneLayout *planes, uint32_t R, hipStream_t stream) {
    // largest tap table, in bytes, that fits the LDS left by the region, if chunks
    // of R records may have it there
    auto table = [&](size_t region) {
        size_t most = 0;
        for (int p = prm.p_lo; p < prm.p_hi; ++p) {
            const size_t w = (size_t)prm.beta * planes[p].S;
            const size_t t = w * w * (SEP ? sizeof(float) : 2 * sizeof(TapT));
            if (region + t <= kWindowLds && R >= stage_records((uint32_t)prm.beta))
                most = std::max(most, t);
        }
        return (most + 7) & ~size_t(7);
    };
    // LDS region of the window gridders: 8 planes of the instance's fixed
    // stride (tile plus the class's largest halo)
    if (cls <= 2 && (tile != kWindowTile || smax > window_smax(cls == 0 ? 1 : cls == 1 ? 4 : 8)))
        return hipErrorInvalidValue;
    switch (cls) {
    case 0: launch_window<1, 1, 8, SEP, TapT>(a, prm, table(window_lds(1)), stream); break;
    case 1: {
        const size_t t = table(window_lds(4));
        if (t == 0)
            launch_window<4, 1, 4, SEP, TapT>(a, prm, 0, stream);
        else
            launch_window<4, 1, 8, SEP, TapT>(a, prm, t, stream);
        break;
    }
    case 2: launch_window<8, 2, 8, SEP, TapT>(a, prm, 0, stream); break;
    default:
        if (region_blocks(tile, smax) > 7 * 16) return hipErrorInvalidValue;
        launch_block<7, 16, SEP, TapT>(a, prm, stream);
        break;
    }
    return hipGetLastError();
}

template <bool SEP>
hipError_t launch_class_t(mg_dtype dt, int cls, const GridPtrs &a, const GridParams &prm,
                          int smax, int tile, const PlaneLayout *planes, uint32_t R,
                          hipStream_t stream) {
    switch (dt) {
    case MG_F16: return launch_class<SEP, __half>(cls, a, prm, smax, tile, planes, R, stream);
    case MG_BF16: return launch_class<SEP, __hip_bfloat16>(cls, a, prm, smax, tile, planes, R, stream);
    default: return launch_class<SEP, float>(cls, a, prm, smax, tile, planes, R, stream);
    }
}

}  // namespace

namespace {
template <typename F>
size_t walk_grid_scratch(const PlanState &P, F &&place) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += arena_round(bytes);
        return at;
    };
    place(0, take(sizeof(float4) * 2 * (size_t)(P.nrec + kRecPad)));
    place(1, take(sizeof(int32_t) * (size_t)P.max_chunks));
    place(2, take(sizeof(uint32_t) * (size_t)P.nplanes_eff));
    return off;
}
}  // namespace

size_t grid_scratch_bytes(const PlanState &P) {
    return walk_grid_scratch(P, [](int, size_t) {});
}

mg_status launch_grid(const PlanState &P, const void *vis, void *grid, void *scratch,
                      hipStream_t stream, const double *factor) {
    if (P.nrec == 0) return MG_OK;
    hipError_t e = hipSuccess;
    void *own = nullptr;
    if (!scratch) {
        e = scratch_alloc(&own, grid_scratch_bytes(P), stream);
        if (e != hipSuccess) return set_error(MG_ENOMEM, "grid: scratch allocation failed");
        scratch = own;
    }
    GridScratch gs;
    walk_grid_scratch(P, [&](int what, size_t at) {
        void *p = static_cast<char *>(scratch) + at;
        if (what == 0) gs.svis = static_cast<float4 *>(p);
        else if (what == 1) gs.uinfo = static_cast<int32_t *>(p);
        else gs.queues = static_cast<uint32_t *>(p);
    });
    const int np = P.nplanes_eff;
    const bool sep = P.kind == MG_KERNEL_SEPARABLE;
    // sorted, scaled visibilities and unit words
    GroupList groups{};
    const int ngroups = plane_groups(P.planes, groups);
    const int gather_groups = (int)std::min<int64_t>(
        resident_groups((const void *)gather_units_kernel, kGatherThreads, 0), P.nrec);
    hipLaunchKernelGGL(gather_units_kernel, dim3(gather_groups, ngroups), dim3(kGatherThreads), 0,
                       stream, P.d_planes, groups, (int32_t)sep, gs.queues, P.bucket_cfirst,
                       P.units, P.group_nunits, P.chunks, P.sperm, (const float2 *)vis,
                       P.geom.npol, factor, gs.svis, gs.uinfo);
    GridPtrs a{P.smeta,   gs.svis,        (float *)grid, P.taps,   P.chunks, P.bucket_cfirst,
               P.units,   P.group_nunits, P.d_planes,   gs.uinfo, nullptr};
    GridParams prm{P.geom.npol, P.geom.nu, P.geom.nv, P.geom.beta, 0, 0,
                   (uint32_t)P.geom.conj_base, 0};
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
        const int cls = P.planes[p0].cls;
        a.queue = gs.queues + p0;
        e = sep ? launch_class_t<true>(P.tap_dtype, cls, a, prm, smax, P.planes[p0].T,
                                       P.planes.data(), (uint32_t)P.R, stream)
                : launch_class_t<false>(P.tap_dtype, cls, a, prm, smax, P.planes[p0].T,
                                        P.planes.data(), (uint32_t)P.R, stream);
        p0 = p1;
    }
    if (e == hipSuccess) e = hipGetLastError();
    if (own) scratch_free(own, stream);
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("grid kernels: ") + hipGetErrorString(e));
    return MG_OK;
}

}  // namespace mg
