// Backward aggregation, column-sliced pull (Eq. 2 right; Eq. 3): a second form of the pull over CSC.
//
// The plain pull gathers whole dY rows on every XCD, so the eight 4 MB L2 caches hold the same 4 thousand rows (dim 256).
// Here a row is cut into slices of one 128-byte cache line (32 fp32 columns, 64 of a 16-bit format) and an XCD works on
// its own slices only: each L2 holds 32 thousand rows of ITS slice, and graphs up to that many source rows - or whose
// entries mostly come from that many - are gathered from L2.  Per (item, slice) the kernel adds up the slice of the
// destination's in-entries in registers (8 lanes x 16 bytes cover one line, so a wave instruction gathers 8 entries) and
// samples the sum at the destination's columns that lie in the slice, through LDS.  Columns may come in any order.
//
// Work: an item longer than kSlicedLongItem is walked by a whole wavefront, its entries in eight equal shares; shorter
// items (the lists are ordered by length) eight to a wavefront, one per group of 8 lanes.  Lane q of a group fetches
// entry q of the group's next eight; quad-wide lane permutes hand (row offset, weight) round, which costs no LDS and
// folds into the address add.  Lanes without an entry gather from an offset past the buffer, which returns 0 and moves
// nothing, so a batch of eight gathers is one run of loads without branches.
//
// What bounds it: the L1 keeps at most 256 lines in flight, which at L2 latency is 0.27 lines per clock per CU (2.1 M
// entries, 4 k nodes, dim 256: 104 us for 17 M lines); beyond L2 the fabric.  Measured us against plain pull (fp32,
// dim 256): 16 k nodes, degree 40, k=128: 57 / 85; 40 k nodes, degree 120, k=128: 362 / 613; 100 k nodes, degree 400,
// k=128: 3462 / 4933; bf16 dY, 60 k nodes, degree 240, k=64: 535 / 820; dim 101, 100 k nodes, degree 60, k=50: 275 / 482.
// Plain pull wins where rows come from beyond L2 anyway (600 k nodes, degree 40, k=64: 4007 / 3198: eight scattered
// lines cost more there than one whole row) and at small k, where it touches fewer lines.
#pragma once

#include <algorithm>

#include "common.hpp"
#include "sspmm_bwd_impl.hpp"

namespace maxk {

// implemented once per storage format of dY (sspmm_bwd_f32.hip, _bf16.hip, _f16.hip)
template <int VT>
maxk_status bwd_sliced_format(const ItemList& L, const int32_t* csc_src, const float* csc_val, const void* dY,
                              const void* sp_index, int index_bytes, int64_t N, int dim, int k, char* copy, float* dXs,
                              float* partials, hipStream_t s);

namespace {

constexpr int kSlicedWaves = 4;  // wavefronts of a workgroup; they share nothing but the launch

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct SlicedArgs {
    const WorkItem* items;  // longest first; the first n_long are walked by whole wavefronts
    const int32_t* src;     // CSC: source row and weight of every in-entry
    const float* val;
    const char* rows;       // dY, or its slice-major copy
    const void* sp_index;
    float* dXs;
    float* partials;
    int64_t slice_stride;   // bytes from a row's slice to its next one
    uint32_t row_stride;    // bytes from a row's slice to the next row's
    uint32_t bytes;         // extent of slice 0; slice s ends slice_shrink * s earlier
    uint32_t slice_shrink;
    uint32_t n_items, n_long, tasks;  // tasks: wavefronts' worth of items
    uint32_t parts, units_per_xcd, wgs_per_unit;
    int32_t dim, k;
};

// lane U of the caller's quad
template <int U>
__device__ __forceinline__ uint32_t quad_lane(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, U * 0x55, 0xF, 0xF, true);
}

// the first / last four lanes of every eight, in both quads of the eight (row_shr:4 into the odd quads resp. row_shl:4
// into the even ones)
__device__ __forceinline__ uint32_t lower_four(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x114, 0xF, 0xA, false);
}
__device__ __forceinline__ uint32_t upper_four(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x104, 0xF, 0x5, false);
}

// sum = w * x for the first entry of a sum, sum += w * x for the others
template <int VT, bool FIRST, int N>
__device__ __forceinline__ void sliced_fma(float (&sum)[N], float w, u32x4 x)
{
    const uint32_t d[4] = {x.x, x.y, x.z, x.w};
    const auto add = [&](float& to, float v) { to = FIRST ? w * v : to + w * v; };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (VT == MAXK_VALUE_F32) {
            add(sum[i], __uint_as_float(d[i]));
        } else {
            add(sum[2 * i], widen_value<VT>((uint16_t)(d[i] & 0xFFFFu)));
            add(sum[2 * i + 1], widen_value<VT>((uint16_t)(d[i] >> 16)));
        }
    }
}

// VEC: consecutive sp_index entries fetched with one load (4 or 1), for the short items.
// fp32 in registers for 8 wavefronts a SIMD (66 registers otherwise: the first shape below 1370 us instead of 1232); the
// 16-bit formats as they come (74 registers, 6 wavefronts: 617 us; held to 8 they spill: 1090).
template <int VT, int VEC, typename IdxT>
__global__ __launch_bounds__(kSlicedWaves * kWave, VT == MAXK_VALUE_F32 ? 8 : 1) void bwd_sliced_kernel(SlicedArgs a)
{
    constexpr int EPL = VT == MAXK_VALUE_F32 ? 4 : 8;  // columns per lane
    constexpr int W = 8 * EPL;                         // columns of a slice
    __shared__ __attribute__((aligned(16))) float lds[kSlicedWaves * 8 * W];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // Workgroup b runs on XCD b % 8.  A unit is one slice and one `parts`-th of the tasks; an XCD takes consecutive
    // units, so it stays on one slice as long as there is one for each XCD.
    const uint32_t b = blockIdx.x >> 3, ul = b / a.wgs_per_unit, unit = (blockIdx.x & 7u) * a.units_per_xcd + ul;
    const uint32_t slice = unit / a.parts, part = unit - slice * a.parts;
    const uint32_t task = ((b - ul * a.wgs_per_unit) * a.parts + part) * kSlicedWaves + wave;
    if (task >= a.tasks) return;
    const int q = lane & 7, g = lane >> 3;
    const bool whole = task < a.n_long;  // wave-uniform
    const int c0 = (int)slice * W, width = min(W, a.dim - c0);
    float* __restrict__ sums = lds + wave * (8 * W);
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(a.rows + (int64_t)slice * a.slice_stride), (short)0, (int)(a.bytes - slice * a.slice_shrink), 0x00020000);

    const uint32_t item = whole ? task : a.n_long + (task - a.n_long) * 8 + g;
    const bool have = item < a.n_items;
    WorkItem it = {0, 0, 0, -1};
    if (whole) it = a.items[__builtin_amdgcn_readfirstlane(item)];
    else if (have) it = a.items[item];
    int p = it.begin, e = it.end;
    if (whole) {
        const int share = (e - p + 7) >> 3;
        p += g * share;
        e = min(e, p + share);
    }
    const uint32_t lane_off = (uint32_t)q * 16u;
    // Entries are added up in fours, which go to two running sums in turn.  One running sum over all entries of a lane group
    // came out up to twice as far from 64 bits as the kernels whose calls come here (runs of 64 entries, 2-norm: 1.4e-7 with
    // one sum, 7.4e-8 so, plain pull 6.8e-8 .. 8.7e-8, expand/reduce 7.1e-8 .. 1.1e-7; of 16: 7.4e-8, 5.6e-8, 5.6e-8 and
    // 6.0e-8).  us, one sum / fours: fp32 60 k nodes, degree 240, k = 64 1223 / 1232; 100 k, degree 60, dim 101, k = 50
    // 332 / 335; bf16 60 k, degree 240, k = 64 627 / 617.
    float first[EPL], second[EPL], four[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) first[i] = second[i] = 0.f;

    constexpr uint32_t kNowhere = 0xFFFF0000u;  // past every buffer (kSlicedMaxBytes), also with lane_off added
    int n = e - p;                              // entries left of this group; <= 0: none
    const auto entry = [&](int at) { return max(min(at + q, e - 1), 0); };  // in range whatever n is (nnz >= 1)
    int32_t row = a.src[entry(p)];
    float weight = a.val[entry(p)];
    while (__any(n > 0)) {
        u32x4 x[8];
        const uint32_t off = q < n ? (uint32_t)row * a.row_stride : kNowhere;
        const uint32_t w = q < n ? __float_as_uint(weight) : 0u;
        const uint32_t off_0 = lower_four(off), w_0 = lower_four(w);
#define MAXK_SLICED_LOAD(H, U) \
    x[H * 4 + U] = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)(quad_lane<U>(off_##H) + lane_off), 0, 0);
#define MAXK_SLICED_FMA(H, U) sliced_fma<VT, U == 0>(four, __uint_as_float(quad_lane<U>(w_##H)), x[H * 4 + U]);
        if (!__any(n > 4)) {  // the last four or fewer
            MAXK_SLICED_LOAD(0, 0) MAXK_SLICED_LOAD(0, 1) MAXK_SLICED_LOAD(0, 2) MAXK_SLICED_LOAD(0, 3)
            MAXK_SLICED_FMA(0, 0) MAXK_SLICED_FMA(0, 1) MAXK_SLICED_FMA(0, 2) MAXK_SLICED_FMA(0, 3)
#pragma unroll
            for (int i = 0; i < EPL; ++i) first[i] += four[i];
            break;
        }
        const uint32_t off_1 = upper_four(off), w_1 = upper_four(w);
        MAXK_SLICED_LOAD(0, 0) MAXK_SLICED_LOAD(0, 1) MAXK_SLICED_LOAD(0, 2) MAXK_SLICED_LOAD(0, 3)
        MAXK_SLICED_LOAD(1, 0) MAXK_SLICED_LOAD(1, 1) MAXK_SLICED_LOAD(1, 2) MAXK_SLICED_LOAD(1, 3)
        p += 8;
        n -= 8;
        row = a.src[entry(p)];
        weight = a.val[entry(p)];
        MAXK_SLICED_FMA(0, 0) MAXK_SLICED_FMA(0, 1) MAXK_SLICED_FMA(0, 2) MAXK_SLICED_FMA(0, 3)
#pragma unroll
        for (int i = 0; i < EPL; ++i) first[i] += four[i];
        MAXK_SLICED_FMA(1, 0) MAXK_SLICED_FMA(1, 1) MAXK_SLICED_FMA(1, 2) MAXK_SLICED_FMA(1, 3)
#pragma unroll
        for (int i = 0; i < EPL; ++i) second[i] += four[i];
#undef MAXK_SLICED_LOAD
#undef MAXK_SLICED_FMA
    }

    // each group's sums -> LDS (the wavefront's own part: its LDS operations execute in program order), then the
    // destination's columns that lie in the slice
#pragma unroll
    for (int i = 0; i < EPL; i += 4)
        *reinterpret_cast<float4*>(sums + g * W + q * EPL + i) =
            make_float4(first[i] + second[i], first[i + 1] + second[i + 1], first[i + 2] + second[i + 2], first[i + 3] + second[i + 3]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (!have) return;
    const int k = a.k;
    float* __restrict__ out = it.slot < 0 ? a.dXs + (int64_t)it.row * k : a.partials + (int64_t)it.slot * k;
    const IdxT* __restrict__ cols = (const IdxT*)a.sp_index + (int64_t)it.row * k;
    if (whole) {
        for (int t = lane; t < k; t += kWave) {
            const int c = (int)cols[t] - c0;
            if ((unsigned)c < (unsigned)width) {
                const float* __restrict__ v = sums + c;  // the eight groups' shares
                out[t] = ((v[0] + v[W]) + (v[2 * W] + v[3 * W])) + ((v[4 * W] + v[5 * W]) + (v[6 * W] + v[7 * W]));
            }
        }
        return;
    }
    const float* __restrict__ mine = sums + g * W;
    for (int t = q * VEC; t < k; t += 8 * VEC) {
        IdxPack<IdxT, VEC> ix;
        ix.load(cols + t);
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const int c = ix.get(i) - c0;
            if ((unsigned)c < (unsigned)width) out[t + i] = mine[c];
        }
    }
}

// Slice-major copy of dY: slice s of row i at ((s * N + i) * 128) bytes, columns past dim are 0.  One 16-byte piece a lane.
template <int VT>
__global__ __launch_bounds__(256) void slice_rows_kernel(const value_store_t<VT>* __restrict__ dY, int64_t N, int dim,
                                                         int n_slices, int vec, u32x4* __restrict__ out)
{
    constexpr int EPL = VT == MAXK_VALUE_F32 ? 4 : 8;
    const int pieces = n_slices * 8;
    const int64_t total = N * pieces, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const int64_t row = i / pieces;
        const int piece = (int)(i - row * pieces), c = piece * EPL;
        union { u32x4 v; value_store_t<VT> e[EPL]; } x;
        x.v = u32x4{0u, 0u, 0u, 0u};
        if (vec) {  // dim % EPL == 0, dY 16-byte aligned
            if (c < dim) x.v = *reinterpret_cast<const u32x4*>(dY + row * dim + c);
        } else {
#pragma unroll
            for (int j = 0; j < EPL; ++j)
                if (c + j < dim) x.e[j] = dY[row * dim + c + j];
        }
        out[((int64_t)(piece >> 3) * N + row) * 8 + (piece & 7)] = x.v;
    }
}

template <int VT>
maxk_status sliced_format(const ItemList& L, const int32_t* csc_src, const float* csc_val, const void* dY,
                          const void* sp_index, int index_bytes, int64_t N, int dim, int k, char* copy, float* dXs,
                          float* partials, hipStream_t s)
{
    constexpr int vb = (int)sizeof(value_store_t<VT>), EPL = 16 / vb;
    const int n_slices = sliced_slices(dim, vb);
    SlicedArgs a{};
    if (copy) {
        const int64_t pieces = N * n_slices * 8;
        hipLaunchKernelGGL((slice_rows_kernel<VT>), dim3((unsigned)std::min<int64_t>((pieces + 255) / 256, 1 << 20)), dim3(256),
                           0, s, (const value_store_t<VT>*)dY, N, dim, n_slices, dim % EPL == 0 && aligned(dY, 16),
                           reinterpret_cast<u32x4*>(copy));
        MAXK_LAUNCH_CHECK();
        a.rows = copy;
        a.row_stride = 128;
        a.slice_stride = N * 128;
        a.bytes = (uint32_t)(N * 128);
    } else {
        a.rows = (const char*)dY;
        a.row_stride = (uint32_t)(dim * vb);
        a.slice_stride = 128;
        a.bytes = (uint32_t)(N * (int64_t)dim * vb);
        a.slice_shrink = 128;
    }
    a.items = L.d_items; a.src = csc_src; a.val = csc_val; a.sp_index = sp_index; a.dXs = dXs; a.partials = partials;
    a.dim = dim; a.k = k;
    a.n_items = (uint32_t)L.n_items;
    a.n_long = (uint32_t)L.n_long;
    a.tasks = (uint32_t)(L.n_long + (L.n_items - L.n_long + 7) / 8);
    int common = 8;  // gcd(n_slices, 8): the slices are dealt to the XCDs in equal parts
    while (n_slices % common) common /= 2;
    a.parts = (uint32_t)(8 / common);
    a.units_per_xcd = (uint32_t)(n_slices * a.parts / 8);
    a.wgs_per_unit = ((a.tasks + kSlicedWaves - 1) / kSlicedWaves + a.parts - 1) / a.parts;
    const int64_t blocks = (int64_t)8 * a.units_per_xcd * a.wgs_per_unit;
    if (blocks > 0xFFFFFFFFll / (kSlicedWaves * kWave)) return MAXK_UNSUPPORTED;  // a launch holds below 2^32 work items
    const bool vec = k % 4 == 0 && aligned(sp_index, 4 * (size_t)index_bytes);
#define MAXK_SLICED(VEC, IDX) \
    hipLaunchKernelGGL((bwd_sliced_kernel<VT, VEC, IDX>), dim3((unsigned)blocks), dim3(kSlicedWaves * kWave), 0, s, a)
    if (index_bytes == 1) { if (vec) MAXK_SLICED(4, uint8_t); else MAXK_SLICED(1, uint8_t); }
    else if (index_bytes == 2) { if (vec) MAXK_SLICED(4, uint16_t); else MAXK_SLICED(1, uint16_t); }
    else { if (vec) MAXK_SLICED(4, int32_t); else MAXK_SLICED(1, int32_t); }
#undef MAXK_SLICED
    MAXK_LAUNCH_CHECK();
    return MAXK_OK;
}

}  // namespace
}  // namespace maxk
