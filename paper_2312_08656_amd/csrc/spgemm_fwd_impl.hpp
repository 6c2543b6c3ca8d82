// Forward aggregation: row-wise-product SpGEMM with dense output
// (Eq. 2 left; Sec. 3.2 "Forward Computation"; prior art: Alg. 1).
//
// One 64-lane wavefront owns one work item (a run of at most `chunk` stored entries of one row of A) or a bin of them, and
// works on 64 / LANES entries side by side, LANES lanes an entry (FwdLanes).  The other k run spgemm_fwd_rmw_kernel, which walks a
// FLAT list of units (entry e, position t), 64 at a time: unit u belongs to entry u / k and CBSR position u % k.
//
// Bound by instruction issue before, by LDS now: a wave instruction of 64 positions took 14 to 20 vector instructions (the entry's
// node and weight, 64-bit addresses, predicates) beside an LDS read-add-write pair of 12 clocks, 8 of them bank conflicts of
// random columns; now it takes 4 to 8: offsets are 32 bits and the broadcasts of an entry's node, row and weight are part of the
// instructions that use them, whole batches need no predicates, and the loads of the next batch's first entries are under way while a
// batch is added.  us, before / now: 2.1 M entries on 4 k nodes, k = 16 29.8 / 21.9; 1.2 M on 40 k, width 100, k = 13 45.3 / 26.7; 4 M on
// 40 k, k = 24 110 / 64; 14.7 M on 717 k, width 384, k = 96 1080 / 957; 115 M on 233 k, k = 32 2025 / 1665, bf16 k = 64 2922 / 2455.
//
// Accumulation.  LDS floating-point atomics (ds_add_f32) retire about one lane
// every three clocks on this chip (measured: ~190 clocks per wave instruction),
// which capped the first version of this kernel at ~200 G updates/s no matter
// the memory system.  A plain LDS read-add-write pair is ~14x faster, and it is
// safe here without atomics because (a) the k positions of one CBSR row are
// distinct columns, and (b) the entries that share one wave instruction (at most
// NB = ceil(64/k)+1 consecutive ones) accumulate into NB PRIVATE copies of the
// output row (copy e % NB; one for each lane group), while LDS operations of one wavefront execute in
// program order.  The copies are added up when the row is written out.
// Rows longer than `chunk` write partial rows that a second kernel adds up
// (deterministic order, and it bounds the length of any fp32 running sum);
// every other row is written once, straight from LDS, fully coalesced.
// Shapes whose private copies would not fit comfortably in LDS (tiny k with a
// very wide row) fall back to the single-copy kernel with LDS atomics.
//
// This header holds the kernel templates; one translation unit per storage format of the CBSR values
// (fp32, bf16, fp16) instantiates them, so the three compile side by side.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "lanes.hpp"

namespace maxk {

// Private output-row copies needed so that entries sharing a wave instruction never collide.
__host__ __device__ constexpr int private_copies(int k)
{
    return (k >= kWave) ? ((k % kWave == 0) ? 1 : 2) : ((kWave % k == 0) ? kWave / k : (kWave - 1) / k + 2);
}

constexpr size_t kMaxPrivateLds = 40 * 1024;  // above this the private copies cost too much occupancy

// Floats between the end of one private copy and the start of the next (a multiple of 4).  Padding shifts the copies
// against each other in the LDS banks; measured without effect (the columns of different entries are unrelated, so
// their bank conflicts are those of random addresses), hence 0.
#ifndef MAXK_FWD_COPY_PAD
#define MAXK_FWD_COPY_PAD 0
#endif
constexpr int kCopyPad = MAXK_FWD_COPY_PAD;

// implemented once per storage format (spgemm_fwd_f32.hip, _bf16.hip, _f16.hip)
template <int VT>
maxk_status launch_fwd_format(const ItemList& L, const int32_t* col, const float* val, const void* sp_data,
                              const void* sp_index, int index_bytes, int64_t N, char* packed, int dim, int k,
                              float* Y, float* partials, hipStream_t s);

template <int VT>
maxk_status launch_fwd_sweep_format(const SweepSet& S, const void* sp_data, const void* sp_index, int index_bytes, int64_t N,
                                    char* packed, int dim, int k, float* Y, float* partials, hipStream_t s);

namespace {


constexpr int kRounds = 4;  // unit rounds in flight per wavefront (fallback kernel)

// Fallback for shapes whose private copies would not fit in LDS: a single copy of the output row,
// updated with LDS floating-point atomics (slow on this chip, see the header comment).
template <int VT, typename IdxT>
__global__ __launch_bounds__(kWave) void spgemm_fwd_atomic_kernel(const WorkItem* __restrict__ items,
                                                                  const int32_t* __restrict__ col,
                                                                  const float* __restrict__ val,
                                                                  const value_store_t<VT>* __restrict__ sp_data,
                                                                  const IdxT* __restrict__ sp_index, int dim, int k,
                                                                  float* __restrict__ Y, float* __restrict__ partials)
{
    extern __shared__ float row_buf[];
    const int lane = threadIdx.x;
    const WorkItem it = items[blockIdx.x];
    for (int c = lane; c < dim; c += kWave) row_buf[c] = 0.f;
    __syncthreads();

    const uint32_t end = it.end;
    for (uint32_t base = it.begin; base < end; base += kWave) {  // (unsigned: the position behind the last entry may pass 2^31)
        const int n = (int)min((uint32_t)kWave, end - base);
        int my_col = 0;
        float my_val = 0.f;
        if (lane < n) {
            my_col = col[base + lane];
            my_val = val[base + lane];
        }
        const int units = n * k;
        for (int u0 = 0; u0 < units; u0 += kWave * kRounds) {
            float d[kRounds], a[kRounds];
            int ix[kRounds];
            bool ok[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int u = u0 + r * kWave + lane;
                ok[r] = u < units;
                const int uc = ok[r] ? u : 0;
                const int e = uc / k;
                const int t = uc - e * k;
                const int c = __shfl(my_col, e);
                a[r] = __shfl(my_val, e);
                const int64_t off = (int64_t)c * k + t;
                d[r] = widen_value<VT>(sp_data[off]);
                ix[r] = (int)sp_index[off];
            }
#pragma unroll
            for (int r = 0; r < kRounds; ++r)
                if (ok[r]) atomicAdd(&row_buf[ix[r]], a[r] * d[r]);
        }
    }
    __syncthreads();

    float* __restrict__ out = (it.slot < 0) ? Y + (int64_t)it.row * dim : partials + (int64_t)it.slot * dim;
    for (int c = lane; c < dim; c += kWave) out[c] = row_buf[c];
}

// A pair: a 16-bit value in the upper half, 4 x its column (below 4096) in the lower one.
__device__ __forceinline__ uint32_t fwd_pair_column(uint32_t p) { return p & 0xFFFFu; }
template <int VT>
__device__ __forceinline__ float fwd_pair_value(uint32_t p)
{
    return VT == MAXK_VALUE_BF16 ? __uint_as_float(p & 0xFFFF0000u) : widen_value<MAXK_VALUE_F16>((uint16_t)(p >> 16));
}

// For small k a CBSR row is a fraction of a cache line in EACH of the two arrays, and the kernel is
// bound by the number of row requests (~137 G/s measured), not by bytes.  The packed path reads a
// per-call repack instead: one record per node, k values followed by k indices, so an entry costs
// one request.  The repack reads and writes N*k*(4+ib) bytes, against nnz*k*(4+ib) for the kernel
// (2+ib with 16-bit values; the indices start at the next multiple of their own width).
template <int LAYOUT, int VT, typename IdxT>
__global__ __launch_bounds__(256) void pack_cbsr_kernel(const value_store_t<VT>* __restrict__ sp_data,
                                                        const IdxT* __restrict__ sp_index, int64_t n_units, int k,
                                                        int rec_bytes, int idx_off, char* __restrict__ packed)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n_units; u += stride) {
        const int64_t node = u / k;
        const int t = (int)(u - node * k);
        char* rec = packed + node * rec_bytes;
        if constexpr (LAYOUT == kFwdPairs) {
            reinterpret_cast<uint32_t*>(rec)[t] = (uint32_t)sp_data[u] << 16 | (uint32_t)sp_index[u] * 4u;
        } else if constexpr (LAYOUT == kFwdHalves) {
            reinterpret_cast<float*>(rec)[t] = sp_data[u];
            reinterpret_cast<uint32_t*>(rec)[8 + t] = (uint32_t)sp_index[u] * 4u;
        } else {
            reinterpret_cast<value_store_t<VT>*>(rec)[t] = sp_data[u];
            reinterpret_cast<IdxT*>(rec + idx_off)[t] = sp_index[u];
        }
    }
}

// ROUNDS: 64-unit rounds in flight;
// PACKED: read the per-node (values, indices) records of pack_cbsr_kernel instead of the two arrays
// VT: storage format of the CBSR values (widened exactly; products and sums are fp32 in every format)
template <int ROUNDS, bool PACKED, int VT, typename IdxT>
__global__ __launch_bounds__(kWave) void spgemm_fwd_rmw_kernel(const WorkItem* __restrict__ items,
                                                               const int32_t* __restrict__ col,
                                                               const float* __restrict__ val,
                                                               const value_store_t<VT>* __restrict__ sp_data,
                                                               const IdxT* __restrict__ sp_index,
                                                               const char* __restrict__ packed, int rec_bytes,
                                                               int idx_off,
                                                               int dim, int k, int nb, int vec_out,
                                                               float* __restrict__ Y, float* __restrict__ partials)
{
    // vec_out: dim % 4 == 0 and Y / partials 16-byte aligned, so that a row is written with 16-byte stores; 2: past
    // L2, but for the partial rows of split ones, which combine_kernel reads next
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int lane = threadIdx.x;
    float* __restrict__ row_buf = lds;                                         // nb copies of the output row
    const int cs = dim + kCopyPad;                                             // floats from one copy to the next
    int2* __restrict__ entry_buf = reinterpret_cast<int2*>(lds + ((nb * cs + 1) & ~1));  // 64 staged (col, val)
    const WorkItem it = items[blockIdx.x];
    if (((nb * cs) & 3) == 0) {
        for (int c = lane * 4; c < nb * cs; c += kWave * 4)
            *reinterpret_cast<float4*>(row_buf + c) = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        for (int c = lane; c < nb * cs; c += kWave) row_buf[c] = 0.f;
    }

    const uint32_t end = it.end;
    for (uint32_t base = it.begin; base < end; base += kWave) {  // (unsigned: the position behind the last entry may pass 2^31)
        const int n = (int)min((uint32_t)kWave, end - base);
        __syncthreads();  // previous batch fully consumed (and the zero fill done)
        if (lane < n) entry_buf[lane] = make_int2(col[base + lane], __float_as_int(val[base + lane]));
        __syncthreads();
        const int units = n * k;
        for (int u0 = 0; u0 < units; u0 += kWave * ROUNDS) {
            float d[ROUNDS], a[ROUNDS];
            int at[ROUNDS];
            bool ok[ROUNDS];
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                const int u = u0 + r * kWave + lane;
                ok[r] = u < units;
                const int uc = ok[r] ? u : 0;
                const int e = uc / k;
                const int t = uc - e * k;
                const int2 ed = entry_buf[e];
                a[r] = __int_as_float(ed.y);
                if constexpr (PACKED) {
                    const char* rec = packed + (int64_t)ed.x * rec_bytes;
                    d[r] = widen_value<VT>(reinterpret_cast<const value_store_t<VT>*>(rec)[t]);
                    at[r] = (e % nb) * cs + (int)reinterpret_cast<const IdxT*>(rec + idx_off)[t];
                } else {
                    const int64_t off = (int64_t)ed.x * k + t;
                    d[r] = widen_value<VT>(sp_data[off]);
                    at[r] = (e % nb) * cs + (int)sp_index[off];
                }
            }
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                if (ok[r]) {
                    const float old = row_buf[at[r]];
                    row_buf[at[r]] = old + a[r] * d[r];
                }
            }
        }
    }
    __syncthreads();

    float* __restrict__ out = (it.slot < 0) ? Y + (int64_t)it.row * dim : partials + (int64_t)it.slot * dim;
    if (vec_out) {
        const bool once = vec_out == 2 && it.slot < 0;
        for (int c = lane * 4; c < dim; c += kWave * 4) {
            float4 acc = *reinterpret_cast<const float4*>(row_buf + c);
            for (int b = 1; b < nb; ++b) {
                const float4 x = *reinterpret_cast<const float4*>(row_buf + b * cs + c);
                acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
            }
            if (once) store_once(out + c, acc); else *reinterpret_cast<float4*>(out + c) = acc;
        }
    } else {
        for (int c = lane; c < dim; c += kWave) {
            float acc = row_buf[c];
            for (int b = 1; b < nb; ++b) acc += row_buf[b * cs + c];
            out[c] = acc;
        }
    }
}


// ---- forward sweep ----
//
// The kernel above has every wavefront gather from its own place in the CBSR, 37 MB of it on the dense workload (k = 32)
// against 4 MB of L2 per XCD: nearly every record comes from beyond L2, and that fabric is what it waits for (7.4 TB/s).
// Here a wavefront keeps a BIN of output rows in LDS and walks the entries of all its rows in the order of their source
// node.  Bins hold about the same number of entries, so the wavefronts resident on an XCD pass over the source nodes at
// about the same pace and share the records they gather through its L2.  As above, entries that share a wave instruction
// add into private copies of the row (one per lane group of K lanes: the same number of partial sums per row), and LDS
// operations of a wavefront execute in order.
//
// A workgroup has half a CU's LDS.  The more rows a wavefront keeps there, the more often a record is met while an L2 holds it: us, rows
// x wavefronts of a workgroup, 115 M entries on 233 k nodes: k = 32 2 x 16 1939, 4 x 10 1755, 5 x 8 1663, 10 x 4 1918 (43 M on 577 k:
// 1250, 1178, 1187, 1179); k = 64 4 x 16 2778, 5 x 16 2626, 10 x 8 2688; k = 128 5 x 16 5470, 10 x 8 4894; k = 16 1 x 16 1293, 2 x 8 1176,
// 4 x 5 1155.  Fetched from beyond L2 at k = 32: 12.2 GB at 2 x 16 (1939 us, the fabric's rate).
// Measured, us, row by row / sweep: 115 M entries on 233 k nodes k = 16 1513 / 1173, k = 32 2774 / 1665, k = 64 5060 / 2633, k = 96 7789 / 5671,
// k = 128 10436 / 4878, bf16 k = 64 3174 / 2455; 79 M entries on 132 k nodes k = 32 1521 / 1109; 43 M on 576 k k = 32
// 1451 / 1216; 126 M on 2.4 M nodes k = 64 5948 / 4490.
//
// The entries are read once and Y is written once: both pass by L2's replacement order and leave its 4 MB to the records.
// us, both plain / so: 43 M entries on 577 k nodes k = 32 1311 / 1276; 126 M on 2.4 M k = 64 4650 / 4547.  Y alone: 115 M on 233 k
// k = 32 2017 / 2005, bf16 k = 64 2935 / 2896; of the kernel above 14.7 M on 717 k, dim 384, k = 96 1169 / 1139; 79 M
// on 133 k k = 8 692 / 682.  Partial rows of split rows are read by the next kernel and stay plain (2.5 M on 169 k k = 32, all plain /
// partial rows past L2 as well / so 89.8 / 91.0 / 89.3).  With a kernel behind it that reads Y the call keeps the gain: 43 M on
// 577 k k = 32 1476 / 1450 for both, 14.7 M on 717 k, dim 384, k = 96 1481 / 1439; rows of 100 or 300 floats too (8.5 M on
// 500 k 336 / 307, 6.2 M on 200 k 286 / 261).
constexpr int kSweepWaves = 16;            // wavefronts of a workgroup, at most
constexpr uint32_t kSweepMeet = 4;         // batches between barriers (5 x 8, k = 32: 1706 / 1681 / 1663 us at 1 / 2 / 4)

// k = 8 from records of 8 fp32 values and 4 x their columns: two groups share 16 lanes, which hold eight entries of each and bring a
// whole record with one load, an access of 64 bytes (values and columns by themselves: two accesses of 32 and 8).
struct FwdHalves : FwdLanes<8, 1> {
    static constexpr int PER = 8, BATCH = 8, HELD = 1;
};

// What one wavefront needs of the CBSR.  Offsets are 32 bits (fwd_wide: the arrays are larger, and they are 64).
// ROWS: the entries say which row of a bin they belong to.
template <class S, int LAYOUT, bool ROWS, int VT, typename IdxT>
struct FwdWave {
    static constexpr bool PAIRS = LAYOUT == kFwdPairs, HALVES = LAYOUT == kFwdHalves, PACKED = LAYOUT != kFwdArrays;
    static_assert(HALVES == std::is_same_v<S, FwdHalves> && (!HALVES || VT == MAXK_VALUE_F32) && (!PAIRS || VT != MAXK_VALUE_F32));
    static constexpr uint32_t kVal = PAIRS ? 4u : sizeof(value_store_t<VT>), kIdx = HALVES ? 4u : sizeof(IdxT);
    using Value = std::conditional_t<PAIRS, uint32_t, value_store_t<VT>>;
    typedef __attribute__((address_space(3))) float lds_float;
    struct Held {  // a batch of entries: node (-1: none) and row; bytes from the first record; LDS bytes of the row; weight
        uint32_t x[S::HELD], d[S::HELD], i[S::HELD], row[S::HELD];
        float w[S::HELD];
    };
    struct Step {
        Value d[S::ROUNDS];
        uint32_t i[PAIRS ? 1 : S::ROUNDS];
    };
    const char* data;
    const char* index;
    uint32_t d_stride, i_stride;             // bytes of a node's values and columns (PACKED: of its record, both)
    uint32_t d_lane, i_lane, d_last, i_last;  // this lane's position in the first and the last pass
    uint32_t own, row_bytes;                  // LDS address of the group's copy; bytes of a row

    __device__ __forceinline__ FwdWave(const value_store_t<VT>* sp_data, const IdxT* sp_index, const char* packed, int rec_bytes, int idx_off,
                                       int dim, int k, int lane, uint32_t group_copy)
    {
        const uint32_t t = (uint32_t)(lane % S::LANES), last = min(t + (uint32_t)((S::PASSES - 1) * S::LANES), (uint32_t)k - 1u);
        data = PACKED ? packed : reinterpret_cast<const char*>(sp_data);
        index = PACKED ? packed + idx_off : reinterpret_cast<const char*>(sp_index);
        d_stride = PACKED ? (uint32_t)rec_bytes : (uint32_t)k * kVal;
        i_stride = PACKED ? (uint32_t)rec_bytes : (uint32_t)k * kIdx;
        d_lane = t * kVal;
        i_lane = t * kIdx;
        d_last = last * kVal;
        i_last = last * kIdx;
        if (HALVES) {  // the first group's record as it is, the second's with its halves changed round
            d_lane = (uint32_t)(lane % 16) * 4u;
            i_lane = d_lane ^ 32u;
        }
        own = group_copy;
        row_bytes = (uint32_t)dim * 4u;
    }

    __device__ __forceinline__ Held hold(const int2 (&e)[S::HELD]) const
    {
        Held h;
#pragma unroll
        for (int r = 0; r < S::HELD; ++r) {
            const uint32_t x = (uint32_t)e[r].x, node = ROWS ? x & ((1u << kSweepRowShift) - 1u) : x;
            const uint32_t n = x == 0xFFFFFFFFu ? 0u : node;  // (padding reads node 0 and drops it)
            h.x[r] = x;
            h.d[r] = n * d_stride;
            h.i[r] = PACKED ? h.d[r] : n * i_stride;
            h.row[r] = ROWS ? own + (x >> kSweepRowShift) * row_bytes : own;
            h.w[r] = __int_as_float(e[r].y);
        }
        return h;
    }

    __device__ __forceinline__ bool gap(const Held& h) const  // whether this lane holds padding
    {
        bool none = false;
#pragma unroll
        for (int r = 0; r < S::HELD; ++r) none |= h.x[r] == 0xFFFFFFFFu;
        return none;
    }

    // Waits for the first loads of a loop.  (Columns that came into it as 8- or 16-bit values would be widened again in every turn.)
    __device__ __forceinline__ void settle(Step& s) const
    {
#pragma unroll
        for (int r = 0; r < (PAIRS || HALVES ? 0 : S::ROUNDS); ++r) asm volatile("" : "+v"(s.i[r]));
    }

    template <int E>
    __device__ __forceinline__ uint32_t entry(const Held& h) const { return held_entry<S::PER, E % S::PER>(h.x[E / S::PER]); }

    // The loads of entries F .. F + STEP - 1
    template <int F, bool WIDE = false, typename Ok>
    __device__ __forceinline__ void load(const Held& h, Step& s, Ok&& ok) const
    {
        const auto one = [&](auto idx) {
            constexpr int R = decltype(idx)::value, E = F + R / S::PASSES, P = R % S::PASSES, H = E / S::PER, I = E % S::PER;
            constexpr bool LAST = !S::WHOLE && P == S::PASSES - 1;
            if (!ok(E)) return;
            if constexpr (HALVES && !WIDE) {
                s.d[R] = *reinterpret_cast<const float*>(data + (uint64_t)(row16_lane<I>(h.d[H]) + d_lane));
                s.i[R] = *reinterpret_cast<const uint32_t*>(data + (uint64_t)(row16_lane<I + 8>(h.d[H]) + i_lane));
                return;
            }
            uint64_t at_d, at_i;
            if constexpr (WIDE) {
                const uint32_t x = held_entry<S::PER, I>(h.x[H]), node = x == 0xFFFFFFFFu ? 0u : ROWS ? x & ((1u << kSweepRowShift) - 1u) : x;
                at_d = (uint64_t)node * d_stride + (LAST ? d_last : d_lane);
                at_i = (uint64_t)node * i_stride + (LAST ? i_last : i_lane);
                if constexpr (HALVES) {
                    const uint32_t x0 = row16_lane<I>(h.x[H]), x1 = row16_lane<I + 8>(h.x[H]), mask = ROWS ? (1u << kSweepRowShift) - 1u : 0xFFFFFFFFu;
                    at_d = (uint64_t)(x0 == 0xFFFFFFFFu ? 0u : x0 & mask) * d_stride + d_lane;
                    at_i = (uint64_t)(x1 == 0xFFFFFFFFu ? 0u : x1 & mask) * d_stride + i_lane;
                }
            } else {
                at_d = held_entry<S::PER, I>(h.d[H]) + (LAST ? d_last : d_lane);
                at_i = held_entry<S::PER, I>(PACKED ? h.d[H] : h.i[H]) + (LAST ? i_last : i_lane);
            }
            constexpr uint32_t skip = LAST ? 0u : (uint32_t)(P * S::LANES);
            s.d[R] = *reinterpret_cast<const Value*>(data + skip * kVal + at_d);
            if constexpr (HALVES) s.i[R] = *reinterpret_cast<const uint32_t*>(data + at_i);
            else if constexpr (!PAIRS) s.i[R] = *reinterpret_cast<const IdxT*>(index + skip * kIdx + at_i);
        };
        [&]<int... I>(std::integer_sequence<int, I...>) { (one(std::integral_constant<int, I>{}), ...); }
        (std::make_integer_sequence<int, S::ROUNDS>{});
    }

    // ... and what they brought, times the weights, into the row.  LDS operations of a wavefront execute in order.
    template <int F, typename Ok>
    __device__ __forceinline__ void add(const Held& h, const Step& s, Ok&& ok) const
    {
        const auto one = [&](auto idx) {
            constexpr int R = decltype(idx)::value, E = F + R / S::PASSES, H = E / S::PER, I = E % S::PER;
            const uint32_t row = ROWS ? held_entry<S::PER, I>(h.row[H]) : own;
            uint32_t column;  // 4 x
            float x;
            if constexpr (PAIRS) {
                column = fwd_pair_column(s.d[R]);
                x = fwd_pair_value<VT>(s.d[R]);
            } else if constexpr (HALVES) {
                const bool low = (threadIdx.x & 8u) == 0;
                const uint32_t first = __float_as_uint(s.d[R]), second = s.i[R];
                x = __uint_as_float(low ? first : second);
                column = (uint32_t)__builtin_amdgcn_mov_dpp((int)(low ? second : first), 0x128, 0xF, 0xF, true);  // from 8 lanes on, round 16
            } else {
                column = s.i[R] * 4u;
                x = widen_value<VT>(s.d[R]);
            }
            lds_float* const at = reinterpret_cast<lds_float*>(row + column);
            const float w = __uint_as_float(held_entry<S::PER, I>(__float_as_uint(h.w[H])));
            if (ok(std::integral_constant<int, E>{})) *at = fmaf(w, x, *at);
        };
        [&]<int... I>(std::integer_sequence<int, I...>) { (one(std::integral_constant<int, I>{}), ...); }
        (std::make_integer_sequence<int, S::ROUNDS>{});
    }
};

// The group's copies of a row, `copy` floats apart, added up and written
template <int GROUPS>
__device__ __forceinline__ void write_out(const float* __restrict__ row, int copy, int dim, int lane, bool vec, bool once, float* __restrict__ out)
{
    if (vec) {
        for (int c = lane * 4; c < dim; c += kWave * 4) {
            float4 acc = *reinterpret_cast<const float4*>(row + c);
#pragma unroll
            for (int g = 1; g < GROUPS; ++g) {
                const float4 x = *reinterpret_cast<const float4*>(row + g * copy + c);
                acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
            }
            if (once) store_once(out + c, acc); else *reinterpret_cast<float4*>(out + c) = acc;
        }
    } else {
        for (int c = lane; c < dim; c += kWave) {
            float acc = row[c];
#pragma unroll
            for (int g = 1; g < GROUPS; ++g) acc += row[g * copy + c];
            out[c] = acc;
        }
    }
}

__device__ __forceinline__ void zero_lds(float* __restrict__ p, int n, int lane)
{
    if ((n & 3) == 0) {
        for (int c = lane * 4; c < n; c += kWave * 4) *reinterpret_cast<float4*>(p + c) = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        for (int c = lane; c < n; c += kWave) p[c] = 0.f;
    }
}

// the wavefront's own LDS, whose operations execute in order: only the compiler has to keep it
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t lds_address(const float* p)
{
    typedef __attribute__((address_space(3))) const float lds_const_float;
    return (uint32_t)(uintptr_t)(lds_const_float*)p;
}

// Row by row: a wavefront per work item.  (k = 8, 10 .. 128 and 192; the others, and some calls at k = 17 .. 21, run spgemm_fwd_rmw_kernel.)
// Wavefronts a SIMD that the registers leave room for: nothing of a pass may spill, and from two passes on 64 registers do not hold two
// sets of loads (two passes of 8 lanes mostly fit).  us, by units / lane groups with spills for 8 wavefronts / with 6: 60 k nodes, degree 16, k = 50 with 4-byte columns
// 82 / 102 / 80, width 512, k = 128 bf16 84 / 108 / 82; 100 k, 61, k = 50 bf16, 2-byte columns 359 / 284 / 231; 300 k, 31, k = 128 786 / 952 / 786.
// Half as many loads under way leave room for more wavefronts, which is better where one group works on an entry (1 M nodes, degree 9,
// k = 128 863 us by units, 1092 with spills, 928 / 854 with all loads / half) and in two passes of 16 lanes (717 k, 11, k = 24 462, 313, 345 / 309),
// but not from column pairs (100 k, 61, k = 24 bf16 89 / 92).
template <class S>
struct HalfStep : S {
    static constexpr int STEP = S::STEP / 2, STEPS = S::BATCH / STEP, ROUNDS = STEP * S::PASSES;
};
template <class S, int LAYOUT>
constexpr bool kRowHalf = (S::LANES == kWave && S::PASSES <= 2) || (S::LANES == 16 && S::PASSES == 2 && LAYOUT != kFwdPairs);
template <class S, int LAYOUT>
using RowSplit = std::conditional_t<kRowHalf<S, LAYOUT>, HalfStep<S>, S>;
template <class S, int LAYOUT, int VT>
constexpr int row_waves()
{
    constexpr bool F32 = VT == MAXK_VALUE_F32;
    if (S::PASSES == 1 || (S::LANES == 8 && S::PASSES == 2 && (F32 || LAYOUT != kFwdArrays))) return 8;
    if (S::LANES == 16 && kRowHalf<S, LAYOUT>) return F32 ? 8 : 7;
    return S::LANES == 8 && S::PASSES == 3 && F32 ? 7 : 6;  // (100 k nodes, degree 17, width 64, k = 17: 55.7 us with 6, 51.8 with 7)
}
template <class S, int LAYOUT, int VT, typename IdxT>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(row_waves<S, LAYOUT, VT>()))) void spgemm_fwd_row_kernel(
    const WorkItem* __restrict__ items, const int32_t* __restrict__ col, const float* __restrict__ val,
    const value_store_t<VT>* __restrict__ sp_data, const IdxT* __restrict__ sp_index, const char* __restrict__ packed, int rec_bytes,
    int idx_off, int dim, int k, int wide, int vec_out, float* __restrict__ Y, float* __restrict__ partials)
{
    extern __shared__ __attribute__((aligned(16))) float row_lds[];
    const int lane = threadIdx.x;
    const WorkItem it = items[blockIdx.x];
    const int copy = (dim + 3) & ~3;  // floats from one copy to the next
    float* __restrict__ row = row_lds;
    zero_lds(row, S::GROUPS * copy, lane);
    wave_lds_fence();
    const int g = lane / S::LANES;
    using Wave = FwdWave<S, LAYOUT, false, VT, IdxT>;
    const Wave wv(sp_data, sp_index, packed, rec_bytes, idx_off, dim, k, lane, lds_address(row + g * copy));
    run_item(wv, EntryBatches<S>(col, val, it.end, lane), it.begin, it.end, g, wide != 0);
    wave_lds_fence();
    float* __restrict__ out = it.slot < 0 ? Y + (int64_t)it.row * dim : partials + (int64_t)it.slot * dim;
    write_out<S::GROUPS>(row, copy, dim, lane, vec_out != 0, vec_out == 2 && it.slot < 0, out);
}

// A workgroup is up to 16 wavefronts with a bin each; they meet at a barrier every kSweepMeet batches, which keeps a CU together on its
// way over the source nodes.
template <class S, int LAYOUT, int VT, typename IdxT>
__global__ __launch_bounds__(kSweepWaves * kWave) __attribute__((amdgpu_waves_per_eu(8))) void spgemm_fwd_sweep_kernel(
    const int2* __restrict__ ent, const uint32_t* __restrict__ batch, const int2* __restrict__ bin_rows, int64_t n_bins,
    int per_bin, const value_store_t<VT>* __restrict__ sp_data, const IdxT* __restrict__ sp_index,
    const char* __restrict__ packed, int rec_bytes, int idx_off, int dim, int k, int wide, int vec_out, float* __restrict__ Y,
    float* __restrict__ partials)
{
    extern __shared__ __attribute__((aligned(16))) float sweep_lds[];
    const int lane = threadIdx.x & (kWave - 1);
    const int waves = blockDim.x / kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t bin0 = (int64_t)blockIdx.x * waves, bin = bin0 + wave;
    const int copy = per_bin * dim, total = S::GROUPS * copy;  // floats of one copy of the bin's rows, and of all of them
    float* __restrict__ rows = sweep_lds + wave * total;
    zero_lds(rows, total, lane);
    wave_lds_fence();
    const uint32_t b0 = bin < n_bins ? batch[bin] : 0u, b1 = bin < n_bins ? batch[bin + 1] : 0u;
    uint32_t longest = 0;  // batches of the workgroup's longest bin: every wavefront meets every barrier
    for (int i = 0; i < waves && bin0 + i < n_bins; ++i) longest = max(longest, batch[bin0 + i + 1] - batch[bin0 + i]);
    const int g = lane / S::LANES;
    using Wave = FwdWave<S, LAYOUT, true, VT, IdxT>;
    const Wave wv(sp_data, sp_index, packed, rec_bytes, idx_off, dim, k, lane, lds_address(rows + g * copy));
    const uint32_t lane_entry = (uint32_t)(g * S::BATCH + lane % S::PER);
    const auto fetch = [&](uint32_t b, int2 (&e)[S::HELD]) {
        const int2* const at = ent + (int64_t)min(b, b1 - 1u) * (S::GROUPS * S::BATCH);
#pragma unroll
        for (int r = 0; r < S::HELD; ++r) e[r] = load_once(at + (lane_entry + (uint32_t)(r * S::PER)));
    };
    const uint32_t n = b1 - b0;
    uint32_t i = 0;
    if (n) {
        int2 e[S::HELD];
        fetch(b0, e);
        typename Wave::Held cur = wv.hold(e);
        fetch(b0 + 1, e);
        const auto there = [&](auto m) { return wv.template entry<decltype(m)::value>(cur) != 0xFFFFFFFFu; };
        if (wide) {
            for (; i < n; ++i) {
                if (i % kSweepMeet == 0) __builtin_amdgcn_s_barrier();
                static_for<S::STEPS>([&](auto j) {
                    typename Wave::Step s;
                    wv.template load<decltype(j)::value * S::STEP, true>(cur, s, kAlways);
                    wv.template add<decltype(j)::value * S::STEP>(cur, s, there);
                });
                cur = wv.hold(e);
                fetch(b0 + i + 2, e);
            }
        } else {
            typename Wave::Step s0, s1;
            wv.template load<0>(cur, s0, kAlways);
            wv.settle(s0);
            const auto batch_of = [&](auto&& ok) {
                typename Wave::Held next;
                static_for<S::STEPS>([&](auto j) {
                    constexpr int J = decltype(j)::value, F = J * S::STEP;
                    typename Wave::Step& now = J % 2 ? s1 : s0;
                    typename Wave::Step& other = J % 2 ? s0 : s1;
                    if constexpr (J + 1 < S::STEPS) {
                        wv.template load<F + S::STEP>(cur, other, kAlways);
                    } else {  // the first ones of the next batch (behind the last: the last batch's again)
                        next = wv.hold(e);
                        wv.template load<0>(next, other, kAlways);
                        fetch(b0 + i + 2, e);
                    }
                    wv.template add<F>(cur, now, ok);
                });
                cur = next;
            };
            // whole batches; the lists of a bin differ by a few entries, so that only its last one or two have gaps
            for (; i < n && __builtin_amdgcn_ballot_w64(wv.gap(cur)) == 0; ++i) {
                if (i % kSweepMeet == 0) __builtin_amdgcn_s_barrier();
                batch_of(kAlways);
            }
            for (; i < n; ++i) {
                if (i % kSweepMeet == 0) __builtin_amdgcn_s_barrier();
                batch_of(there);
            }
        }
    }
    for (; i < longest; ++i)
        if (i % kSweepMeet == 0) __builtin_amdgcn_s_barrier();
    if (bin >= n_bins) return;
    wave_lds_fence();
    for (int r = 0; r < per_bin; ++r) {
        const int2 to = bin_rows[bin * per_bin + r];
        if (to.x < 0) continue;
        float* __restrict__ out = to.y < 0 ? Y + (int64_t)to.x * dim : partials + (int64_t)to.y * dim;
        write_out<S::GROUPS>(rows + r * dim, copy, dim, lane, vec_out != 0, vec_out == 2 && to.y < 0, out);
    }
}

// Runs F<FwdLanes<LANES, PASSES>> for MaxK k.  SWEEP: the sweep takes eight lane groups at k = 8 alone (sweep_takes).
template <int LAYOUT, bool SWEEP, typename F>
maxk_status for_fwd_groups(int k, F&& f)
{
    const FwdGroups by = fwd_groups(k);
    if constexpr (LAYOUT == kFwdHalves) return f.template operator()<FwdHalves>();
    else {
#define MAXK_FWD_GROUPS(LANES, PASSES) \
    if (by.lanes == LANES && by.passes == PASSES) return f.template operator()<FwdLanes<LANES, PASSES>>()
    MAXK_FWD_GROUPS(8, 1);
    MAXK_FWD_GROUPS(16, 1);
    if constexpr (!SWEEP) MAXK_FWD_GROUPS(8, 2);
    if constexpr (!SWEEP && LAYOUT != kFwdPairs) MAXK_FWD_GROUPS(8, 3);
    MAXK_FWD_GROUPS(16, 2);
    MAXK_FWD_GROUPS(32, 1);
    if constexpr (LAYOUT == kFwdArrays) {
        MAXK_FWD_GROUPS(16, 3);
        MAXK_FWD_GROUPS(16, 4);
        MAXK_FWD_GROUPS(32, 3);
        MAXK_FWD_GROUPS(32, 4);
        MAXK_FWD_GROUPS(64, 1);
        MAXK_FWD_GROUPS(64, 2);
        if constexpr (!SWEEP) MAXK_FWD_GROUPS(64, 3);
    }
#undef MAXK_FWD_GROUPS
    return MAXK_UNSUPPORTED;
    }
}

template <int LAYOUT, int VT, typename IdxT>
maxk_status launch_sweep(const SweepSet& S, const value_store_t<VT>* sp_data, const IdxT* sp_index, const char* packed,
                         int rec_bytes, int idx_off, int64_t N, int dim, int k, float* Y, float* partials, hipStream_t s)
{
    const size_t lds = sizeof(float) * (size_t)(S.groups * S.per_bin) * (size_t)dim;
    const int waves = sweep_waves(k, S.per_bin, dim);
    if (waves < 1) return MAXK_UNSUPPORTED;
    const int vec_out = dim % 4 == 0 && aligned(Y, 16) && aligned(partials, 16) ? (past_l2(N * dim * 4) ? 2 : 1) : 0;
    const dim3 grid((unsigned)((S.n_bins + waves - 1) / waves)), block((unsigned)(kWave * waves));
    const int wide = fwd_wide(N, k, (int)sizeof(value_store_t<VT>), (int)sizeof(IdxT), LAYOUT ? rec_bytes : 0);
    return for_fwd_groups<LAYOUT, true>(k, [&]<class G>() -> maxk_status {
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&spgemm_fwd_sweep_kernel<G, LAYOUT, VT, IdxT>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSweepLds);
        MAXK_HIP_TRY(attr);
        hipLaunchKernelGGL((spgemm_fwd_sweep_kernel<G, LAYOUT, VT, IdxT>), grid, block, lds * waves, s, S.d_ent, S.d_batch, S.d_rows, S.n_bins,
                           S.per_bin, sp_data, sp_index, packed, rec_bytes, idx_off, dim, k, wide, vec_out, Y, partials);
        MAXK_LAUNCH_CHECK();
        return MAXK_OK;
    });
}

template <int LAYOUT, int VT, typename IdxT>
maxk_status launch_row(const ItemList& L, const int32_t* col, const float* val, const value_store_t<VT>* sp_data,
                       const IdxT* sp_index, const char* packed, int rec_bytes, int idx_off, int64_t N, int dim, int k, float* Y,
                       float* partials, hipStream_t s)
{
    if (L.n_items > 0x7FFFFFFF) return MAXK_UNSUPPORTED;
    const int vec_out = dim % 4 == 0 && aligned(Y, 16) && aligned(partials, 16) ? (past_l2(N * dim * 4) ? 2 : 1) : 0;
    if (const int lanes = fwd_groups(k).lanes; !fwd_by_units(k, dim, (int)sizeof(value_store_t<VT>), L.n_items, L.n_entries)) {
        const int wide = fwd_wide(N, k, (int)sizeof(value_store_t<VT>), (int)sizeof(IdxT), LAYOUT ? rec_bytes : 0);
        const size_t lds = sizeof(float) * (size_t)(kWave / lanes) * (size_t)((dim + 3) & ~3);
        return for_fwd_groups<LAYOUT, false>(k, [&]<class G>() -> maxk_status {
            hipLaunchKernelGGL((spgemm_fwd_row_kernel<RowSplit<G, LAYOUT>, LAYOUT, VT, IdxT>), dim3((unsigned)L.n_items), dim3(kWave), lds, s, L.d_items, col, val,
                               sp_data, sp_index, packed, rec_bytes, idx_off, dim, k, wide, vec_out, Y, partials);
            MAXK_LAUNCH_CHECK();
            return MAXK_OK;
        });
    }
    if constexpr (LAYOUT == kFwdPairs || LAYOUT == kFwdHalves) return MAXK_UNSUPPORTED;
    else {
        const int nb = private_copies(k);
        const size_t lds = sizeof(float) * (size_t)((nb * (dim + kCopyPad) + 1) & ~1) + sizeof(int2) * kWave;
        hipLaunchKernelGGL((spgemm_fwd_rmw_kernel<8, LAYOUT == kFwdRecord, VT, IdxT>), dim3((unsigned)L.n_items), dim3(kWave), lds, s, L.d_items,
                           col, val, sp_data, sp_index, packed, rec_bytes, idx_off, dim, k, nb, vec_out, Y, partials);
        MAXK_LAUNCH_CHECK();
        return MAXK_OK;
    }
}

// Calls launch(layout, index type's stand-in, record bytes, column offset) on the layout for this call, repacking the CBSR first
// where there is a workspace for it.
template <int VT, typename IdxT, typename F>
maxk_status with_layout(const value_store_t<VT>* sp_data, const IdxT* sp_index, int64_t N, char* packed, int k, hipStream_t s, F&& launch)
{
    const int vb = (int)sizeof(value_store_t<VT>), ib = (int)sizeof(IdxT);
    const int layout = packed ? fwd_layout(k, ib, vb) : kFwdArrays;
    if (layout == kFwdArrays) return launch(std::integral_constant<int, kFwdArrays>{}, sp_index, 0, 0);
    const int rec_bytes = fwd_packed_record_bytes(k, ib, vb), idx_off = fwd_packed_index_offset(k, ib, vb);
    const int64_t n_units = N * (int64_t)k;
    const dim3 blocks((unsigned)std::min<int64_t>((n_units + 255) / 256, 65536));
    const auto repacked = [&](auto l, auto* index, int offset) -> maxk_status {
        hipLaunchKernelGGL((pack_cbsr_kernel<decltype(l)::value, VT, IdxT>), blocks, dim3(256), 0, s, sp_data, sp_index, n_units, k, rec_bytes, idx_off, packed);
        MAXK_LAUNCH_CHECK();
        return launch(l, index, rec_bytes, offset);
    };
    const uint8_t* const any = nullptr;  // (columns of one width)
    if constexpr (VT == MAXK_VALUE_F32) {
        if (layout == kFwdHalves) return repacked(std::integral_constant<int, kFwdHalves>{}, any, 0);
    } else {
        if (layout == kFwdPairs) return repacked(std::integral_constant<int, kFwdPairs>{}, any, 0);
    }
    return repacked(std::integral_constant<int, kFwdRecord>{}, sp_index, idx_off);
}

template <int VT, typename IdxT>
maxk_status launch_sweep_i(const SweepSet& S, const value_store_t<VT>* sp_data, const IdxT* sp_index, int64_t N, char* packed,
                           int dim, int k, float* Y, float* partials, hipStream_t s)
{
    return with_layout<VT>(sp_data, sp_index, N, packed, k, s, [&](auto layout, auto* index, int rec_bytes, int idx_off) {
        return launch_sweep<decltype(layout)::value, VT>(S, sp_data, index, packed, rec_bytes, idx_off, N, dim, k, Y, partials, s);
    });
}

template <int VT>
maxk_status launch_fwd_sweep_vt(const SweepSet& S, const void* sp_data_v, const void* sp_index, int index_bytes, int64_t N,
                                char* packed, int dim, int k, float* Y, float* partials, hipStream_t s)
{
    const auto* sp_data = (const value_store_t<VT>*)sp_data_v;
    if (index_bytes == 1) return launch_sweep_i<VT>(S, sp_data, (const uint8_t*)sp_index, N, packed, dim, k, Y, partials, s);
    if (index_bytes == 2) return launch_sweep_i<VT>(S, sp_data, (const uint16_t*)sp_index, N, packed, dim, k, Y, partials, s);
    return launch_sweep_i<VT>(S, sp_data, (const int32_t*)sp_index, N, packed, dim, k, Y, partials, s);
}

template <int VT, typename IdxT>
maxk_status launch_atomic(const ItemList& L, const int32_t* col, const float* val, const value_store_t<VT>* sp_data,
                          const IdxT* sp_index, int dim, int k, float* Y, float* partials, hipStream_t s)
{
    if (L.n_items > 0x7FFFFFFF) return MAXK_UNSUPPORTED;
    hipLaunchKernelGGL((spgemm_fwd_atomic_kernel<VT, IdxT>), dim3((unsigned)L.n_items), dim3(kWave),
                       sizeof(float) * (size_t)dim, s, L.d_items, col, val, sp_data, sp_index, dim, k, Y, partials);
    MAXK_LAUNCH_CHECK();
    return MAXK_OK;
}

template <int VT, typename IdxT>
maxk_status launch_row_i(const ItemList& L, const int32_t* col, const float* val, const value_store_t<VT>* sp_data,
                         const IdxT* sp_index, int64_t N, char* packed, int dim, int k, float* Y, float* partials,
                         hipStream_t s)
{
    return with_layout<VT>(sp_data, sp_index, N, packed, k, s, [&](auto layout, auto* index, int rec_bytes, int idx_off) {
        return launch_row<decltype(layout)::value, VT>(L, col, val, sp_data, index, packed, rec_bytes, idx_off, N, dim, k, Y, partials, s);
    });
}

// everything but the final sum of split rows, for one storage format of the values
template <int VT>
maxk_status launch_fwd_vt(const ItemList& L, const int32_t* col, const float* val, const void* sp_data_v,
                          const void* sp_index, int index_bytes, int64_t N, char* packed, int dim, int k, float* Y,
                          float* partials, hipStream_t s)
{
    const auto* sp_data = (const value_store_t<VT>*)sp_data_v;
    const bool units = fwd_by_units(k, dim, (int)sizeof(value_store_t<VT>), L.n_items, L.n_entries);
    const size_t private_lds = sizeof(float) * (size_t)(units ? private_copies(k) : kWave / fwd_groups(k).lanes) * (size_t)dim;
    if (private_lds <= kMaxPrivateLds) {
        if (index_bytes == 1) return launch_row_i<VT>(L, col, val, sp_data, (const uint8_t*)sp_index, N, packed, dim, k, Y, partials, s);
        if (index_bytes == 2) return launch_row_i<VT>(L, col, val, sp_data, (const uint16_t*)sp_index, N, packed, dim, k, Y, partials, s);
        return launch_row_i<VT>(L, col, val, sp_data, (const int32_t*)sp_index, N, packed, dim, k, Y, partials, s);
    }
    if (index_bytes == 1) return launch_atomic<VT>(L, col, val, sp_data, (const uint8_t*)sp_index, dim, k, Y, partials, s);
    if (index_bytes == 2) return launch_atomic<VT>(L, col, val, sp_data, (const uint16_t*)sp_index, dim, k, Y, partials, s);
    return launch_atomic<VT>(L, col, val, sp_data, (const int32_t*)sp_index, dim, k, Y, partials, s);
}

}  // namespace
}  // namespace maxk
