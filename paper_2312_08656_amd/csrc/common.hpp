// Internal declarations shared by the translation units of libmaxk (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/maxk.h"

namespace maxk {

constexpr int kWave = 64;  // CDNA wavefront width

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Streams that a kernel reads or writes once pass by the L2's replacement order, so that the records it gathers stay.
// Forward output below the size of the eight L2s together is better left there: its way out would add to the end of a short kernel
// (forward, 2.1 M entries on 4 k nodes 28.1 us plain / 29.0; 1.2 M on 40 k 40.0 / 40.9; 169 k nodes, 173 MB of Y 99.9 / 98.9).
inline bool past_l2(int64_t bytes) { return bytes > (32 << 20); }

// The products of expand/reduce, which one kernel writes and the next one reads.  They pass by L2 where they do not fit the
// Infinity Cache (256 MiB) with the rest of the pass: entries, dY, columns, result, and H, Y and dH around the call.  Within it the
// plain ones come back from there and a store past L2 only delays them.  The two kernels alone, us, plain / past L2, width 256: 4 k nodes,
// 0.3 M entries, k = 128 69 / 91; 6 k nodes, k = 32 70 / 81 (205 MB of products), 118 / 99 (260); 150 k, k = 32 132 / 114 (120); alone the
// sides cross at 236 to 286 MB of what the call itself touches (14 series of graphs), below 40 MB of products they are within 3 us.  A whole pass
// (with kernels behind it that read Y and dH): 25 k nodes, k = 16, 42 MB of products 67.3 / 69.0 (84.0 / 86.0); 40 k, k = 32, 128 MB 108.5 / 111.2
// (152.9 / 141.2), 164 MB 136.5 / 126.5 (176 / 156); 117 k, k = 16, 157 MB 285 / 278 (376 / 392).  Product rows that are not whole 64-byte
// sectors share them, and they then move twice (1.7 M entries, 45 k nodes, k = 13 92 / 123; 25 M on 592 k, k = 8 1109 / 1142).
constexpr double kInfinityCache = 256.0 * (1 << 20);
inline bool products_past_l2(int64_t N, int64_t nnz, int dim, int k, int index_bytes, int val_bytes)
{
    return k % 16 == 0 && (double)nnz * (4.0 * k + 12.0) + (double)N * (dim * (val_bytes + 12.0) + (4.0 + index_bytes) * k) > kInfinityCache;
}

// The rows that the gradient scatter writes.  Past L2 from 32 MiB up where they are whole 64-byte sectors: the kernel by itself
// gains above the Infinity Cache only and is up to 33 % slower below it where k is small, but the pass around it keeps H, Y
// and dY closer.  us of a whole pass, plain / past L2 (with kernels behind it that read Y and dH): 169 k nodes, width 256, k = 32 440 / 422
// (556 / 540); 117 k, k = 16 295 / 278 (397 / 392); 78 k, width 384, k = 96 479 / 463 (563 / 557); 133 k, k = 8 1710 / 1702 (1810 /
// 1801); 59 k, k = 16 133.5 / 133.9 (191.5 / 190.3).  Other rows share their sectors, which then move twice, up to 1.6 times
// the kernel's time; only larger ones gain over the pass: width 300, 60 MB 227 / 228 (274 / 276), 190 MB 755 / 753 (895 / 887), 320 MB
// 1304 / 1294; width 500, 60 MB 138 / 136 (183 / 188), 120 MB 265 / 263 (350 / 354), 190 MB 416 / 407; width 260, 60 MB 281 / 284
// (324 / 329), 190 MB 870 / 872 (988 / 988); width 100, 60 MB 338 / 333 (380 / 381), 190 MB 1147 / 1131.
inline bool scatter_past_l2(int64_t N, int dim) { return (double)N * dim * 4.0 > (dim % 16 == 0 ? 32.0 * (1 << 20) : 160e6); }
__device__ __forceinline__ void store_once(float* p, float4 x)
{
    __builtin_nontemporal_store(f32x4{x.x, x.y, x.z, x.w}, reinterpret_cast<f32x4*>(p));
}
__device__ __forceinline__ float4 load_once(const float4* p)
{
    const f32x4 x = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    return make_float4(x.x, x.y, x.z, x.w);
}
__device__ __forceinline__ int2 load_once(const int2* p)  // 8 bytes, aligned
{
    const uint64_t x = __builtin_nontemporal_load(reinterpret_cast<const uint64_t*>(p));
    return make_int2((int)(uint32_t)x, (int)(uint32_t)(x >> 32));
}

// One unit of scheduled work: a contiguous run of stored entries of one row
// (forward / push backward / dense SpMM) or of one column of A^T (pull backward).
// The paper's "edge group" (Sec. 4.1), sized for a 64-wide wavefront.
struct WorkItem {
    int32_t row;    // output row (or destination node for the CSC lists)
    int32_t begin;  // first stored entry
    int32_t end;    // one past the last
    int32_t slot;   // -1: this item owns the whole row and writes the result; else partial-sum slot
};

// First entry of the batch at position `base` of the entries of a work item that ends at `end`: the item's last entry where the batch lies
// behind it.  Positions are unsigned: batches are fetched two ahead, and an item may end at 2^31 - 16.
__host__ __device__ constexpr uint32_t batch_begin(uint32_t base, uint32_t end) { return base < end ? base : end - 1u; }

// A row whose entries were split over several items; its partial sums live in
// slots [slot_begin, slot_begin + slot_count) and are added up by a second kernel.
struct SplitRow {
    int32_t row;
    int32_t slot_begin;
    int32_t slot_count;
};

struct ItemList {
    WorkItem* d_items = nullptr;
    SplitRow* d_split = nullptr;
    int64_t n_items = 0;
    int64_t n_split = 0;
    int64_t n_slots = 0;
    int64_t n_entries = 0;
    int64_t n_long = 0;  // items longer than kSlicedLongItem entries (they come first: longest first)
};

// The column-sliced pull walks items longer than this with a whole wavefront (8 entries at a time) and shorter ones with
// 8 lanes each (16 / 32 / 64 measured within 3 % of each other, 64 best on graphs of 40 k nodes and more)
constexpr int kSlicedLongItem = 64;

// The visits of a slab that the row-accumulating kernel gives a wavefront each: the first `count` of its long ones, of more
// than `over` entries.
struct LoneVisits { int32_t over, count; };

// A^T regrouped for the L2-tiled pull kernel: source rows are cut into slabs of `slab_rows`
// rows (a slab of dY fits one XCD's L2); in-entries are ordered by (slab of source, destination,
// source) and every non-empty (slab, destination) pair is one "visit".
struct SlabSet {
    int32_t slab_rows = 0;
    int32_t n_slabs = 0;
    int64_t n_visits = 0;
    int32_t* d_src = nullptr;          // [nnz] source row of each regrouped in-entry
    float* d_val = nullptr;            // [nnz]
    int32_t* d_visit_node = nullptr;   // [n_visits] destination node
    int32_t* d_visit_begin = nullptr;  // [n_visits + 1] first regrouped entry of the visit
    int64_t* h_slab_visit = nullptr;   // host [n_slabs + 1] first visit of each slab
    // visits with more than kSlabLongVisit entries (hub destinations) are worked on by a whole wavefront
    int64_t n_long = 0;
    int32_t* d_long_visit = nullptr;   // [n_long] visit numbers, grouped by slab
    int64_t* h_slab_long = nullptr;    // host [n_slabs + 1] first long visit of each slab
    LoneVisits* h_slab_lone = nullptr; // host [n_slabs]
};

constexpr int kSlabLongVisit = 32;

// A^T regrouped for the LDS-tiled backward kernel: destinations are cut into sets of D nodes (a workgroup keeps one
// set's accumulators in LDS), sources into tiles of TR rows; every non-empty (tile, destination) pair is a visit,
// listed per (destination set, tile) and padded to whole wave instructions of E visits.
struct TiledSet {
    int32_t D = 0, TR = 0, E = 0, LPV = 0;  // destinations per set; rows per tile; visits per wave instruction; lanes per visit
    int32_t n_dsets = 0, n_tiles = 0;
    int32_t G = 0, R = 0, tiles_per_range = 0;  // destination sets per XCD; source ranges; tiles per range
    int32_t ovf_by_bucket = 0;                  // overflow entries: added bucket by bucket (1) or with LDS atomics (0)
    int64_t total_sets = 0, n_visits = 0, n_chain = 0;
    uint32_t* d_dir_sets = nullptr;  // [n_dsets * n_tiles + 1 (+ spare)] first wave instruction of each list
    uint2* d_rec = nullptr;          // [total_sets * E] visit records (first entry inline)
    uint4* d_extra = nullptr;        // [total_sets * E] second and third entry of a visit
    uint4* d_ovf = nullptr;          // [n_chain + 1] fourth and later entries of a visit (added at the end of the kernel)
    uint32_t* d_ovf_dir = nullptr;   // [n_dsets * R * lane groups + 1] overflow entries before every (workgroup, lane group)
    uint32_t* d_progress = nullptr;  // [8 * ceil(n_dsets / 8) * 32] progress marks of the running workgroups (pacing)
};

// A^T regrouped for the register-tiled backward kernel (sspmm_bwd_regs.hip).  The head of the destinations, most in-entries first, is
// dealt to sets; a workgroup holds the accumulators of a set in its registers and takes the source rows that the set has
// entries from through LDS, a tile at a time.  A step is a tile and up to kRegsListRecords records for each wavefront.
constexpr int kRegsWaves = 8;            // wavefronts of a workgroup, one workgroup a CU
constexpr int kRegsListRecords = 32;     // 16-byte records (two entries each) of a wavefront's list in one step
constexpr int kRegsTileBuffers = 3;
constexpr int kRegsSpareSteps = 4;       // headers behind the last step, which the kernel reads
constexpr int regs_slots(int kr) { return kr == 2 ? 55 : 111; }  // destinations (per lane group) of a wavefront; one more takes the padding
struct RegsLayout { int rows, head; };   // rows that a wavefront brings per step; 4-byte words of its header
constexpr RegsLayout regs_layout(int pitch)
{
    return pitch == 256 ? RegsLayout{24, 32} : pitch == 512 ? RegsLayout{12, 16} : pitch == 1024 ? RegsLayout{6, 8} : pitch == 1536 ? RegsLayout{4, 8} : RegsLayout{3, 8};
}
constexpr int regs_batch_records(int groups, int kr) { return kr == 2 ? 1 : groups == 1 ? 2 : 4; }  // a list is whole batches
// What a wavefront with `records` records from `record0` on in a tile works on in the tile's step i.  The kernel copies at least one
// record a step: where the list has ended (another wavefront's is longer), record 0, which is always there.
struct RegsStepList { uint32_t first, records; };
__host__ __device__ constexpr RegsStepList regs_step_list(uint32_t record0, uint32_t records, uint32_t i)
{
    const uint32_t done = i * (uint32_t)kRegsListRecords;
    if (done >= records) return {0u, 0u};
    return {record0 + done, records - done < (uint32_t)kRegsListRecords ? records - done : (uint32_t)kRegsListRecords};
}
constexpr uint32_t regs_copied(uint32_t records) { return records > 1u ? records : 1u; }
struct RegsUnit { int32_t set, begin, end, part_begin, part_end; };  // steps [begin, end) of a set, and its parts (none: the set is one part)
struct RegsSum { int32_t set, whole_begin, whole_end, hot_begin, hot_end; };  // the parts of a set in which all slots leave, and the others
struct RegsSplit { int32_t node, row_begin, row_end; };  // a destination that is several ones: their rows of `extra`
struct RegsPart { int32_t end, slots; int64_t at; };  // step behind its last; the sums of that many slots leave then, kRegsHotSlots or all; where to
// Destinations are dealt to slots most in-entries first: the sums of the first slots get long first.
constexpr int kRegsHotSlots = 16;  // (a multiple of the four registers that leave at a time)
struct RegsShape {
    int32_t pitch = 0, groups = 0, kr = 0;  // bytes of a row in LDS; destinations that share a register; registers a destination
    int32_t n_sets = 0, spread = 0;         // sets; sets that a run of destinations is dealt over (1: sets by falling degree)
    int32_t ranges = 0;                     // units a set (0: by cost)
    int32_t run = 0;                        // entries that a destination adds up before its sum leaves the registers, about (0: a unit's)
    int32_t longest = 0;                    // entries that it may at most (0: as many as it has)
    int64_t cap = 0;                        // in-entries of a destination above which it is several ones, with every n-th entry each
    int64_t head = 0;                       // destinations in the sets; the others have the fewest in-entries
    bool operator==(const RegsShape&) const = default;
};
struct RegsSet {
    RegsShape shape;
    int64_t n_units = 0, n_steps = 0, n_records = 0;
    uint4* d_rec = nullptr;
    uint32_t* d_hdr = nullptr;
    int32_t* d_node = nullptr;     // destination of every accumulator, or -1
    int32_t* d_row = nullptr;      // the row its sum goes to: of dXs, from N on of `extra`
    float* d_extra = nullptr;
    int64_t extra_floats = 0;
    RegsSplit* d_split = nullptr;
    int64_t n_split = 0, n_tail = 0;  // destinations that are several ones; destinations behind the head
    RegsUnit* d_unit = nullptr;
    RegsPart* d_part = nullptr;
    float* d_parts = nullptr;      // partial sums of sets in several parts (a call's workspace)
    int64_t n_parts = 0, part_floats = 0, hot_parts = 0;  // the parts in which only the first slots leave begin at hot_parts
    RegsSum* d_sum = nullptr;      // the sets in several parts
    int64_t n_sums = 0;
};

// A regrouped for the forward sweep kernel: work items are dealt to bins of per_bin output rows with about the same number
// of entries; a wavefront keeps a bin's rows in LDS and walks the entries of all of them in the order of their source node.
// Entry e of a row goes to lane group (e + place of the row in the bin) % groups; a batch holds the next sweep_batch(k)
// entries of each group.
struct SweepSet {
    int32_t groups = 0, batch_len = 0, per_bin = 0;
    int64_t n_bins = 0;
    int2* d_ent = nullptr;         // {source node | row of the bin << kSweepRowShift, or -1 (padding); weight}
    uint32_t* d_batch = nullptr;   // [n_bins + 1] first batch of every bin
    int2* d_rows = nullptr;        // [n_bins * per_bin] {output row or -1, partial-sum slot or -1}
};
constexpr int kSweepRowShift = 26, kSweepMaxRows = 31;  // source nodes below 2^26, at most 31 rows a bin

// Where a wavefront finds a node's values and columns: in the two arrays, or in the node's record - columns behind values; 16-bit
// values each with its column, which one load of 4 bytes brings; 8 fp32 values and, as words, 4 x their columns.
enum : int { kFwdArrays = 0, kFwdRecord = 1, kFwdPairs = 2, kFwdHalves = 3 };

// Lanes of an entry and wave instructions an entry in the kernels that work by lane groups (lanes = 0: the others run).  As many
// groups as there were private copies, so that a row has no fewer partial sums, and of those the fewest idle lanes.
struct FwdGroups { int lanes, passes; };
constexpr FwdGroups fwd_groups(int k)
{
    if (k == 64 || k == 128 || k == 192) return {64, k / 64};
    if (k == 8 || k == 16 || k == 32) return {k, 1};
    if (k < 10 || k > 128) return {0, 0};
    if (k <= 21) return {8, (k + 7) / 8};
    if (k <= 63) return {16, (k + 15) / 16};
    return {32, (k + 31) / 32};
}

// Whether the row-by-row kernel works by units (spgemm_fwd_rmw_kernel).  k = 17 to 21 by lane groups has eight copies of a row to clear and to
// add up, by units five: more than it gains where rows are wide and items short.  us, by units / lane groups, fp32: 60 k nodes, degree 16, width
// 256 k = 17 48.4 / 44.6, 384 50.4 / 53.6, 512 60.8 / 71.2; 40 k, 31, width 1024 123 / 151; 1 M, 9, width 384 834 / 893; 300 k, 31, width 512
// 484 / 513; 100 k, 61, width 512 226 / 200, 1024 401 / 433.  bf16: 60 k, 16, width 384 61.3 / 61.5, 512 71.9 / 79.4; 1 M, 9, width 384 916 / 867;
// 300 k, 31, width 512 456 / 413; 40 k, 31, width 1024 136 / 145.
constexpr bool fwd_by_units(int k, int dim, int val_bytes, int64_t items, int64_t entries)
{
    return !fwd_groups(k).lanes ||
           (k >= 17 && k <= 21 && dim > (val_bytes == 4 ? 256 : 384) && entries * (val_bytes == 4 ? 9 : 18) < items * dim);
}

// Whether byte offsets into the CBSR need more than 32 bits (record: bytes of a packed one, 0: two arrays)
inline int fwd_wide(int64_t N, int k, int val_bytes, int index_bytes, int record)
{
    return N * (record ? (int64_t)record : (int64_t)k * std::max(val_bytes, index_bytes)) > 0xFFFFFFFFll;
}
int fwd_layout(int k, int index_bytes, int val_bytes);  // of a repacked CBSR

// k that the sweep takes.  Eight groups in two or three passes lost to the row-by-row kernel on every graph measured (k = 12: eight copies of a
// row leave a bin one row).
constexpr bool sweep_takes(int k) { return fwd_groups(k).lanes && k <= 128 && (fwd_groups(k).lanes > 8 || k == 8); }
constexpr int sweep_groups(int k) { return kWave / fwd_groups(k).lanes; }
constexpr int sweep_batch(int k) { return fwd_groups(k).lanes < 16 ? 8 : 16; }

// LDS of a workgroup of the sweep, two on a CU, its wavefronts, and the rows of a bin.  The rows follow k, and the width only below
// 129 columns, so that most widths walk one regrouped A; more rows where they are short, fewer wavefronts where they are long: us,
// rows 2 / 5 / 10: k = 32, 30 M entries on 300 k nodes, dim 128 708 / 670 / 609; 60 M on 300 k, dim 64 5 / 10 / 20 rows 1184 / 860 / 860; 45 M
// on 150 k, dim 512 842 / 853 / -; k = 96, dim 384 2832 / 2263 (row by row 2960); k = 128, dim 512 5 / 10 rows 3274 / 2385 (4645).
constexpr int64_t kSweepLds = 80 * 1024;
constexpr int sweep_bin_rows(int k, int dim)
{
    const int groups = sweep_groups(k), base = groups == 8 ? 1 : groups == 4 ? 2 : groups == 2 || k == kWave ? 5 : 10;
    const int rows = base * (dim <= 64 ? 4 : dim <= 128 ? 2 : 1);
    return rows < kSweepMaxRows ? rows : kSweepMaxRows;
}
constexpr int sweep_waves(int k, int per_bin, int dim)  // 0: a bin does not fit
{
    const int64_t room = kSweepLds / ((int64_t)sweep_groups(k) * per_bin * dim * 4), most = k == kWave ? 16 : 8;
    return (int)(room < most ? room : most);
}

extern thread_local int32_t g_last_hip_error;

inline maxk_status hip_fail(hipError_t e)
{
    g_last_hip_error = (int32_t)e;
    (void)hipGetLastError();  // clear the sticky launch error, the code is kept above
    return e == hipErrorOutOfMemory ? MAXK_OUT_OF_MEMORY : MAXK_HIP_ERROR;
}

#define MAXK_HIP_TRY(expr)                                   \
    do {                                                     \
        hipError_t _e = (expr);                              \
        if (_e != hipSuccess) return ::maxk::hip_fail(_e);   \
    } while (0)

#define MAXK_LAUNCH_CHECK()                                  \
    do {                                                     \
        hipError_t _e = hipGetLastError();                   \
        if (_e != hipSuccess) return ::maxk::hip_fail(_e);   \
    } while (0)

// ---- storage formats of CBSR values: MAXK_VALUE_F32 / _BF16 / _F16 (the 16-bit ones are bit patterns in uint16_t) ----

template <int VT>
struct value_store { using type = uint16_t; };
template <>
struct value_store<MAXK_VALUE_F32> { using type = float; };
template <int VT>
using value_store_t = typename value_store<VT>::type;

inline int value_bytes(int value_type) { return value_type == MAXK_VALUE_F32 ? 4 : 2; }

// the fp32 value a stored pattern stands for (exact)
template <int VT>
__device__ __forceinline__ float widen_value(value_store_t<VT> x)
{
    if constexpr (VT == MAXK_VALUE_F32) return x;
    else if constexpr (VT == MAXK_VALUE_BF16) return __uint_as_float((uint32_t)x << 16);
    else return (float)__builtin_bit_cast(_Float16, x);
}

// round to nearest, halfway cases to even; beyond the largest finite value -> infinity (NaN is outside the contract)
template <int VT>
__device__ __forceinline__ value_store_t<VT> narrow_value(float x)
{
    if constexpr (VT == MAXK_VALUE_F32) return x;
    else if constexpr (VT == MAXK_VALUE_BF16) {
        const uint32_t b = __float_as_uint(x);
        // adding 0x7FFF (+1 when the kept part is odd) carries into the kept part exactly when the cut-off
        // part is above one half, or equals one half next to an odd neighbour
        return (uint16_t)((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
    } else {
        return __builtin_bit_cast(uint16_t, (_Float16)x);  // v_cvt_f16_f32, round-to-nearest-even mode, subnormals kept
    }
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// ---- launchers implemented in the kernel files (device pointers throughout) ----

maxk_status launch_topk(const float* H, int64_t N, int dim, int k, void* sp_data, int value_type, void* sp_index,
                        int index_bytes, hipStream_t s);

maxk_status launch_cbsr_scatter(const float* values, const void* sp_index, int index_bytes, int64_t N, int dim, int k,
                                float* dense, hipStream_t s);

// `packed`: workspace of N * fwd_packed_record_bytes(k, index_bytes, value bytes) bytes to use the packed-record
// path, or null
maxk_status launch_spgemm_fwd(const ItemList& items, const int32_t* col, const float* val, const void* sp_data,
                              int value_type, const void* sp_index, int index_bytes, int64_t N, char* packed, int dim,
                              int k, float* Y, float* partials, hipStream_t s);
// the same on a regrouped A (fwd_groups(k).lanes > 0, sweep_groups(k) == sweep.groups)
maxk_status launch_spgemm_fwd_sweep(const ItemList& items, const SweepSet& sweep, const void* sp_data, int value_type,
                                    const void* sp_index, int index_bytes, int64_t N, char* packed, int dim, int k, float* Y,
                                    float* partials, hipStream_t s);
int fwd_packed_index_offset(int k, int index_bytes, int val_bytes);  // where a record's indices start
int fwd_packed_record_bytes(int k, int index_bytes, int val_bytes);
int fwd_private_copies(int k);  // output-row copies the forward kernel keeps for MaxK k

maxk_status launch_spmm(const ItemList& items, const int32_t* col, const float* val, const float* H, int dim,
                        float* Y, float* partials, hipStream_t s);

// backward launchers: `dY` holds value_store_t<value_type> elements (fp32, or bf16 / fp16 patterns)
maxk_status launch_bwd_pull(const ItemList& csc_items, const int32_t* csc_src, const float* csc_val, const void* dY,
                            int value_type, const void* sp_index, int index_bytes, int64_t N, int dim, int k, bool units, float* dXs,
                            float* partials, hipStream_t s);

// Column-sliced pull: slices of one 128-byte line of a dY row.  It gathers from dY itself when rows are whole lines and
// 16-byte aligned, else from a slice-major copy made by the call (`copy`, sliced_copy_bytes; odd rows would straddle one
// line more per slice).  Offsets are 32 bits: each slice must end within kSlicedMaxBytes.  MAXK_UNSUPPORTED: too many
// work items for one launch (nothing was launched but the copy).
constexpr int64_t kSlicedMaxBytes = 0xFFFF0000ll;
inline int sliced_slices(int dim, int val_bytes) { return (dim * val_bytes + 127) / 128; }
inline bool sliced_in_place(int dim, int val_bytes) { return dim * val_bytes % 128 == 0; }
inline bool sliced_supports(const void* dY, int64_t N, int dim, int val_bytes)
{
    return sliced_in_place(dim, val_bytes) ? aligned(dY, 16) && N * (int64_t)dim * val_bytes <= kSlicedMaxBytes
                                           : N * 128 <= kSlicedMaxBytes;
}
inline int64_t sliced_copy_bytes(int64_t N, int dim, int val_bytes) { return N * 128 * sliced_slices(dim, val_bytes); }
maxk_status launch_bwd_sliced(const ItemList& csc_items, const int32_t* csc_src, const float* csc_val, const void* dY,
                              int value_type, const void* sp_index, int index_bytes, int64_t N, int dim, int k, char* copy,
                              float* dXs, float* partials, hipStream_t s);

maxk_status launch_bwd_push(const ItemList& items, const int32_t* col, const float* val, const void* dY,
                            int value_type, const void* sp_index, int index_bytes, int64_t N, int dim, int k,
                            float* dXs, hipStream_t s);

// once: the products pass by L2
maxk_status launch_bwd_expand_reduce(const ItemList& csr_items, const int32_t* col, const float* val,
                                     const ItemList& csc_items, const uint32_t* csc_entry, const void* dY,
                                     int value_type, const void* sp_index, int index_bytes, int dim, int k, bool once,
                                     float* expand, float* dXs, float* partials, hipStream_t s);

maxk_status launch_bwd_slab_pull(const SlabSet& S, const void* dY, int value_type, const void* sp_index,
                                 int index_bytes, int64_t N, int dim, int k, float* dXs, hipStream_t s);

// LDS-tiled backward kernel (fp32 dY, k % 4 == 0, dim % 4 == 0, dim <= 512)
struct TiledShape { int D = 0, TR = 0, n_dsets = 0, R = 0; };  // R: source ranges
bool tiled_shape(int64_t N, int64_t nnz, int dim, int k, TiledShape& sh);  // false: (N, dim, k) not supported
int tiled_positions_per_lane(int k);
bool tiled_supports(const void* dY, int value_type, const void* sp_index, int index_bytes, int dim, int k);
maxk_status build_tiled(TiledSet& T, int64_t N, int64_t nnz, const int32_t* d_csc_ptr, const int32_t* d_csc_src,
                        const float* d_csc_val, int D, int TR, int k);
void free_tiled(TiledSet& T);
maxk_status launch_bwd_tiled(const TiledSet& T, const void* dY, int value_type, const void* sp_index, int index_bytes,
                             int64_t N, int dim, int k, float* dXs, hipStream_t s);

bool regs_fits(int dim, int val_bytes, int k, RegsShape& sh);  // pitch, groups and kr; false: (dim, format, k) not supported
maxk_status build_regs(RegsSet& T, const RegsShape& shape, int64_t N, int64_t nnz, const int32_t* d_rowptr, const int32_t* d_csc_ptr, const int32_t* d_csc_src,
                       const float* d_csc_val);
void free_regs(RegsSet& T);
maxk_status launch_bwd_regs(const RegsSet& T, const void* dY, int value_type, const void* sp_index, int index_bytes, int64_t N, int dim,
                            int k, float* dXs, hipStream_t s);
template <int VT>
maxk_status launch_regs_format(const RegsSet& T, const void* dY, const void* sp_index, int index_bytes, int64_t N, int dim, int k, float* dXs,
                               hipStream_t s);

// shared by the push and slab kernels: p[0..n) = 0
maxk_status launch_fill_zero(float* p, int64_t n, hipStream_t s);

// out[row,:] = sum of the row's partial slots, for every split row (width = row length in floats)
maxk_status launch_combine(const ItemList& items, const float* partials, int width, float* out, hipStream_t s);

}  // namespace maxk
