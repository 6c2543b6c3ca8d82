// Backward aggregation, register-tiled form (Eq. 2 right; Eq. 3; prior art: Alg. 2's staging of a dY row on chip): building its
// tables, and adding up what leaves the registers.  The kernel is in sspmm_bwd_regs_impl.hpp.
//
// A workgroup (one per CU, 8 wavefronts) owns a set of destination nodes, keeps their accumulators in its VECTOR REGISTERS -
// 112 a lane beside 112 with their columns, of the 512 KB a CU has - and takes the source rows that the set has entries from
// through LDS, 48 rows of 1 KB a step, by copies that need no register (global_load_lds).  Per entry it then reads the row
// at the destination's columns from LDS and adds to registers: an accumulator's number is taken from the entry's record and
// added to the register numbers of an instruction (VGPR index mode).  Against accumulators in LDS (sspmm_bwd_tiled.hip) that
// leaves one LDS access of three an entry, no read-add-write for the next entry to wait for, and twice the destinations a
// workgroup, so half the rows to bring; against the pull kernels a row is brought once per set instead of once per entry.
// us, before / now, width 256 unless said (115 M entries on 233 k nodes): k = 32 4760 / 2405 (tiled), k = 64 5380 / 3570 and bf16 dY
// 3970 / 2825 (slab pull), k = 128 6270 / 5355; 126 M on 2.4 M nodes, k = 64 14870 / 6560 (pull); 14.7 M directed on 717 k, width 384,
// k = 96 2385 / 1593 (pull); 43 M on 576 k, k = 32 2770 / 2382 (expand/reduce).
//
// Sets.  Destinations are sorted by in-entries, so that a wavefront's lists are about equal.  With as many even sets as CUs, all
// CUs sweep the rows in step and an XCD brings a row into its L2 once; where a set uses few of the rows (large sparse
// graphs) sets by falling degree use fewer of them: 0.35 a stored entry on the graph of 2.4 M nodes, 0.24 to 0.45 on the others.
// Rounding.  A sum in a register is one running sum, so it leaves the register several times a sweep ("parts", kept as they
// are and added up in 64 bits by a second kernel): after `run` entries by a set's mean, and in no case after more than `longest`,
// which is counted when the tables are built.  Nothing is added with atomics: a call gives the same bits every time.
#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include <rocprim/rocprim.hpp>

#include "common.hpp"

namespace maxk {
namespace {

constexpr double kRegsMaxParts[2] = {64.0, 32.0};  // of a set: for the first slots, and for all
constexpr double kRegsUnitCost = 2000.0;  // a unit by cost: about 200 us, against some 25 to begin and end one
constexpr uint32_t kNowhere = 0xFFFFFFFFu;  // place of a destination that is in no set

// a destination's place: accumulator | lane group << 8 | wavefront << 10 | set << 13
__host__ __device__ constexpr uint32_t place_of(uint32_t acc, uint32_t group, uint32_t wave, uint32_t set)
{
    return acc | group << 8 | wave << 10 | set << 13;
}

__global__ __launch_bounds__(256) void regs_degree_kernel(const int32_t* __restrict__ ptr, int64_t N, uint32_t* __restrict__ degree,
                                                          int32_t* __restrict__ node)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    degree[j] = (uint32_t)(ptr[j + 1] - ptr[j]);
    node[j] = (int32_t)j;
}

// A destination of more than `cap` in-entries is several ones (a "share" each); most are one.  shares[j], and a list of those that are several.
__global__ __launch_bounds__(256) void regs_shares_kernel(const int32_t* __restrict__ csc_ptr, int64_t N, int64_t cap, uint32_t* __restrict__ shares,
                                                          uint32_t* __restrict__ count, uint2* __restrict__ several)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j > N) return;
    const int64_t n = j < N ? csc_ptr[j + 1] - csc_ptr[j] : 0, m = n > cap ? (n + cap - 1) / cap : 1;
    shares[j] = j < N ? (uint32_t)m : 0u;
    if (m > 1) several[atomicAdd(count, 1u)] = make_uint2((uint32_t)j, (uint32_t)m);
}

__global__ __launch_bounds__(256) void regs_extra_kernel(const RegsSplit* __restrict__ split, int64_t n, uint32_t* __restrict__ extra0)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) extra0[split[i].node] = (uint32_t)split[i].row_begin;
}

// shares of a destination: in-entries (every m-th one), the destination, and the row that its sum goes to
__global__ __launch_bounds__(256) void regs_share_kernel(const int32_t* __restrict__ csc_ptr, const uint32_t* __restrict__ share0, int64_t N,
                                                         const uint32_t* __restrict__ extra0, uint32_t* __restrict__ degree, int32_t* __restrict__ id,
                                                         int2* __restrict__ goes)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    const uint32_t first = share0[j], m = share0[j + 1] - first, n = (uint32_t)(csc_ptr[j + 1] - csc_ptr[j]);
    for (uint32_t i = 0; i < m; ++i) {
        degree[first + i] = n / m + (i < n % m ? 1u : 0u);
        id[first + i] = (int32_t)(first + i);
        goes[first + i] = make_int2((int32_t)j, (int32_t)(m == 1 ? (uint32_t)j : (uint32_t)N + extra0[j] + i));
    }
}

// Shares in falling order of in-entries are dealt to the lists (set, wavefront, lane group) of `spread` sets forth and
// back, so that the lists of a run of sets have about the same number of entries.
__global__ __launch_bounds__(256) void regs_place_kernel(const int32_t* __restrict__ order, const int2* __restrict__ goes, int64_t n_shares, int64_t head,
                                                         int32_t spread, int32_t groups, int32_t slots, int32_t kr,
                                                         const uint32_t* __restrict__ degree, uint32_t* __restrict__ place,
                                                         int32_t* __restrict__ node, int32_t* __restrict__ row, uint32_t* __restrict__ entries)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= n_shares) return;
    const int32_t v = order[q];
    if (q >= head) {
        place[v] = kNowhere;
        return;
    }
    const int64_t lists = (int64_t)spread * kRegsWaves * groups, run = q / (lists * slots), at = q % (lists * slots);
    const int32_t slot = (int32_t)(at / lists);
    int64_t c = at % lists;
    if (slot & 1) c = lists - 1 - c;
    const int32_t set = (int32_t)(run * spread + c % spread), w = (int32_t)(c / spread) % kRegsWaves, g = (int32_t)(c / spread) / kRegsWaves;
    place[v] = place_of((uint32_t)(slot * kr), (uint32_t)g, (uint32_t)w, (uint32_t)set);
    const int64_t to = ((int64_t)set * kRegsWaves + w) * (slots * groups) + slot * groups + g;
    node[to] = goes[v].x;
    row[to] = goes[v].y;
    entries[to] = degree[q];
}

// rank[] of order[]
__global__ __launch_bounds__(256) void regs_rank_kernel(const int32_t* __restrict__ order, int64_t N, int32_t* __restrict__ rank)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q < N) rank[order[q]] = (int32_t)q;
}

// where[p] = place of the destination of in-entry p; the rows that each set has entries from are marked in `used`
__global__ __launch_bounds__(256) void regs_mark_kernel(const int32_t* __restrict__ csc_ptr, const int32_t* __restrict__ csc_src, int64_t N,
                                                        int64_t nnz, const uint32_t* __restrict__ share0, const uint32_t* __restrict__ place,
                                                        const int32_t* __restrict__ rank, int64_t words,
                                                        uint32_t* __restrict__ where, uint32_t* __restrict__ used)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < nnz; p += stride) {
        int64_t lo = 0, hi = N;  // largest j with csc_ptr[j] <= p
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)csc_ptr[mid] <= p) lo = mid; else hi = mid;
        }
        const uint32_t first = share0[lo], m = share0[lo + 1] - first, at = place[m == 1 ? first : first + (uint32_t)(p - csc_ptr[lo]) % m];
        where[p] = at;
        if (at == kNowhere) continue;
        const int32_t i = rank[csc_src[p]];
        uint32_t* const word = used + ((int64_t)(at >> 13) * words + (i >> 5));
        const uint32_t bit = 1u << (i & 31);
        if (!(*word & bit)) atomicOr(word, bit);
    }
}

__global__ __launch_bounds__(256) void regs_popcount_kernel(const uint32_t* __restrict__ used, int64_t n, uint32_t* __restrict__ count)
{
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (w <= n) count[w] = w < n ? __popc(used[w]) : 0u;
}

// rows[]: the used rows of every set, set after set
__global__ __launch_bounds__(256) void regs_rows_kernel(const uint32_t* __restrict__ used, const uint32_t* __restrict__ before, int64_t n,
                                                        int64_t words, const int32_t* __restrict__ order, uint32_t* __restrict__ rows)
{
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (w >= n) return;
    uint32_t bits = used[w], at = before[w];
    const uint32_t row = (uint32_t)(w % words) * 32u;
    while (bits) {
        rows[at++] = (uint32_t)order[row + (uint32_t)__ffs(bits) - 1u];
        bits &= bits - 1;
    }
}

struct RegsTables {
    const uint32_t* used;
    const uint32_t* before;    // used rows before a word of `used`
    const uint32_t* tile0;     // [sets + 1] first tile of a set
    const int32_t* rank;       // place of a source row in the order that the sets take them in
    int64_t words;
    int32_t tile_rows, pitch, groups, kr;
};

// key: (tile, wavefront, lane group) of an entry's list; what its record says
__global__ __launch_bounds__(256) void regs_keys_kernel(const RegsTables t, const int32_t* __restrict__ csc_src, const float* __restrict__ csc_val,
                                                        const uint32_t* __restrict__ where, int64_t nnz, uint32_t n_lists,
                                                        uint32_t* __restrict__ key, uint2* __restrict__ entry)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < nnz; p += stride) {
        const uint32_t at = where[p];
        if (at == kNowhere) {
            key[p] = n_lists;
            entry[p] = make_uint2(0u, 0u);
            continue;
        }
        const uint32_t set = at >> 13, i = (uint32_t)t.rank[csc_src[p]];
        const int64_t first = (int64_t)set * t.words, w = first + (i >> 5);
        const uint32_t rank = t.before[w] + __popc(t.used[w] & ((1u << (i & 31)) - 1u)) - t.before[first];
        const uint32_t tile = t.tile0[set] + rank / (uint32_t)t.tile_rows, row = rank % (uint32_t)t.tile_rows;
        key[p] = (tile * kRegsWaves + (at >> 10 & 7u)) * (uint32_t)t.groups + (at >> 8 & 3u);
        entry[p] = make_uint2((tile % kRegsTileBuffers * (uint32_t)t.tile_rows + row) * (uint32_t)t.pitch + (at & 0xFFu), __float_as_uint(csc_val[p]));
    }
}

// start[l] = entries in lists below l
__global__ __launch_bounds__(256) void regs_starts_kernel(const uint32_t* __restrict__ key, int64_t nnz, int64_t n_lists, uint32_t* __restrict__ start)
{
    const int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (l > n_lists) return;
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)key[mid] < l) lo = mid + 1; else hi = mid;
    }
    start[l] = (uint32_t)lo;
}

// Records of wavefront w's list of a tile, whole batches: two entries of one list a record, or the e-th entries of the lane groups
__device__ uint32_t regs_list_records(const RegsTables& t, const uint32_t* __restrict__ start, int64_t tile, int w)
{
    const int64_t l = (tile * kRegsWaves + w) * t.groups;
    uint32_t longest = 0;
    for (int g = 0; g < t.groups; ++g) longest = max(longest, start[l + g + 1] - start[l + g]);
    const uint32_t r = t.groups == 1 ? (longest + 1) / 2 : longest * (uint32_t)(t.groups / 2), b = (uint32_t)regs_batch_records(t.groups, t.kr);
    return (r + b - 1) / b * b;
}

__global__ __launch_bounds__(256) void regs_tiles_kernel(const RegsTables t, const uint32_t* __restrict__ start, int64_t n_tiles,
                                                         uint32_t* __restrict__ steps, uint32_t* __restrict__ records)
{
    const int64_t tile = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (tile > n_tiles) return;
    if (tile == n_tiles) {
        steps[tile] = 0;
        records[tile * kRegsWaves] = 0;
        return;
    }
    uint32_t most = 1;
    for (int w = 0; w < kRegsWaves; ++w) {
        const uint32_t r = regs_list_records(t, start, tile, w);
        records[tile * kRegsWaves + w] = r;
        most = max(most, (r + kRegsListRecords - 1) / kRegsListRecords);
    }
    steps[tile] = most;
}

// Headers of a tile's steps for one wavefront, and the longest list of each step (what it costs)
__global__ __launch_bounds__(256) void regs_headers_kernel(const RegsTables t, const uint32_t* __restrict__ start, const uint32_t* __restrict__ rows,
                                                           int64_t n_tiles, int32_t n_sets, int32_t rows_per_wave, int32_t head,
                                                           const uint32_t* __restrict__ step0, const uint32_t* __restrict__ record0,
                                                           uint32_t* __restrict__ hdr, uint8_t* __restrict__ cost,
                                                           uint32_t* __restrict__ pos)
{
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t tile = id / kRegsWaves;
    const int w = (int)(id % kRegsWaves);
    if (tile >= n_tiles) {  // steps behind the last: no list, row 0 into the buffers that are not in use any more
        if (tile < n_tiles + kRegsSpareSteps)
            hdr[((int64_t)step0[n_tiles] + (tile - n_tiles)) * kRegsWaves * head + w * head + 1] = (uint32_t)(tile % kRegsTileBuffers) << 8;
        return;
    }
    int32_t lo = 0, hi = n_sets;  // last set whose first tile is not beyond this one (sets without tiles share theirs with the next)
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if ((int64_t)t.tile0[mid] <= tile) lo = mid; else hi = mid;
    }
    const uint32_t local = (uint32_t)(tile - t.tile0[lo]);
    const int64_t first = (int64_t)lo * t.words;
    const uint32_t row_begin = t.before[first], row_end = t.before[first + t.words];
    const uint32_t records = regs_list_records(t, start, tile, w);
    for (uint32_t s = step0[tile], i = 0; s < step0[tile + 1]; ++s, ++i) {
        const RegsStepList list = regs_step_list(record0[tile * kRegsWaves + w], records, i);
        uint32_t* const h = hdr + ((int64_t)s * kRegsWaves + w) * head;
        h[0] = list.first;
        h[1] = list.records / (uint32_t)regs_batch_records(t.groups, t.kr) | (uint32_t)tile % kRegsTileBuffers << 8;
        for (int r = 0; r < rows_per_wave; ++r) {
            const uint32_t at = row_begin + local * (uint32_t)t.tile_rows + (uint32_t)(w * rows_per_wave + r);
            h[2 + r] = rows[min(at, row_end - 1)];
        }
        if (w == 0) {
            uint32_t longest = 0;
            for (int v = 0; v < kRegsWaves; ++v) longest = max(longest, regs_step_list(0u, regs_list_records(t, start, tile, v), i).records);
            cost[s] = (uint8_t)longest;
            pos[s] = (uint32_t)t.rank[rows[min(row_begin + local * (uint32_t)t.tile_rows, row_end - 1)]];
        }
    }
}

__global__ __launch_bounds__(256) void regs_padding_kernel(uint4* __restrict__ rec, int64_t n, uint32_t spare)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) rec[i] = make_uint4(spare, 0u, spare, 0u);
}

__global__ __launch_bounds__(256) void regs_records_kernel(const RegsTables t, const uint32_t* __restrict__ key, const uint2* __restrict__ entry,
                                                           int64_t n, const uint32_t* __restrict__ start, const uint32_t* __restrict__ record0,
                                                           uint2* __restrict__ rec)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += stride) {
        const uint32_t l = key[p], g = l % (uint32_t)t.groups;
        const int64_t e = p - start[l], first = record0[l / (uint32_t)t.groups];
        rec[first * 2 + (t.groups == 1 ? e : e * t.groups + g)] = entry[p];
    }
}

// Counts, where each sum of a part will be stored, the entries that go into it - of the accumulators that have more than `longest` -
// and notes for every set the largest count above that, of the first slots and of the others.
__global__ __launch_bounds__(256) void regs_longest_kernel(const RegsTables t, const uint32_t* __restrict__ key, const uint2* __restrict__ entry, int64_t n,
                                                           const uint32_t* __restrict__ start, const uint32_t* __restrict__ step0, int32_t n_sets,
                                                           int32_t slots, const uint32_t* __restrict__ entries, const int2* __restrict__ part_range,
                                                           const RegsPart* __restrict__ part, uint32_t longest, uint32_t* __restrict__ count,
                                                           uint32_t* __restrict__ most)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += stride) {
        const uint32_t l = key[p], g = l % (uint32_t)t.groups, w = l / (uint32_t)t.groups % kRegsWaves, tile = l / (uint32_t)t.groups / kRegsWaves;
        int32_t set = 0, hi = n_sets;  // as in regs_headers_kernel
        while (hi - set > 1) {
            const int32_t mid = (set + hi) >> 1;
            if (t.tile0[mid] <= tile) set = mid; else hi = mid;
        }
        const int32_t slot = (int32_t)((entry[p].x & 0xFFu) / (uint32_t)t.kr);
        if (entries[(((int64_t)set * kRegsWaves + w) * slots + slot) * t.groups + g] <= longest) continue;
        const uint32_t e = (uint32_t)p - start[l], record = (t.groups == 1 ? e : e * (uint32_t)t.groups + g) / 2;
        const uint32_t step = step0[tile] + record / (uint32_t)kRegsListRecords;
        int32_t at = part_range[set].x, last = part_range[set].y - 1;  // the first part that ends behind the step
        if (at > last) continue;
        while (at < last) {
            const int32_t mid = (at + last) >> 1;
            if ((uint32_t)part[mid].end > step) last = mid; else at = mid + 1;
        }
        const bool hot = slot < kRegsHotSlots;
        while (!hot && part[at].slots != slots) ++at;  // (the last part of a unit has them all)
        const int64_t to = part[at].at + (((int64_t)w * part[at].slots + slot) * t.kr * kWave + g);
        const uint32_t now = atomicAdd(count + to, 1u) + 1u;
        if (now > longest) atomicMax(most + 2 * set + (hot ? 0 : 1), now);
    }
}

}  // namespace

bool regs_fits(int dim, int val_bytes, int k, RegsShape& sh)
{
    const int row = dim * val_bytes;
    if (row % 16 != 0 || row > 2048 || k < 1 || k > 128) return false;
    sh.pitch = row <= 256 ? 256 : row <= 512 ? 512 : row <= 1024 ? 1024 : row <= 1536 ? 1536 : 2048;
    sh.kr = k > 64 ? 2 : 1;
    sh.groups = k > 32 ? 1 : k > 16 ? 2 : 4;
    return true;
}

void free_regs(RegsSet& T)
{
    (void)hipFree(T.d_rec);
    (void)hipFree(T.d_hdr);
    (void)hipFree(T.d_node);
    (void)hipFree(T.d_row);
    (void)hipFree(T.d_extra);
    (void)hipFree(T.d_split);
    (void)hipFree(T.d_unit);
    (void)hipFree(T.d_part);
    (void)hipFree(T.d_parts);
    (void)hipFree(T.d_sum);
    T = RegsSet();
}

// Synchronises the device.
maxk_status build_regs(RegsSet& T, const RegsShape& shape, int64_t N, int64_t nnz, const int32_t* d_rowptr, const int32_t* d_csc_ptr, const int32_t* d_csc_src,
                       const float* d_csc_val)
{
    const int32_t slots = regs_slots(shape.kr), S = shape.n_sets;
    const RegsLayout layout = regs_layout(shape.pitch);
    const int32_t tile_rows = layout.rows * kRegsWaves;
    const int64_t words = (N + 31) / 32, n_words = words * S, per_set = (int64_t)slots * shape.groups * kRegsWaves;
    if (N < 1 || nnz < 1 || S < 1 || S >= (1 << 19) || shape.head > per_set * S || shape.spread < 1 || S % shape.spread != 0 || n_words > (1 << 29))
        return MAXK_UNSUPPORTED;
    MAXK_HIP_TRY(hipDeviceSynchronize());
    hipStream_t s = nullptr;
    struct Held {  // temporary device memory, given back on every way out
        std::vector<void*> at;
        ~Held() { for (void* p : at) (void)hipFree(p); }
    } held;
    const auto get = [&](auto*& p, int64_t n) {
        p = nullptr;
        held.at.push_back(nullptr);
        const hipError_t e = hipMalloc((void**)&p, sizeof(*p) * (size_t)std::max<int64_t>(n, 1));
        held.at.back() = p;
        return e;
    };
    const auto drop = [&](auto*& p) {
        (void)hipFree(p);
        std::replace(held.at.begin(), held.at.end(), (void*)p, (void*)nullptr);
        p = nullptr;
    };
#define MAXK_TRY_CLEAN(expr)                                                           \
    do {                                                                               \
        const hipError_t _e = (expr);                                                  \
        if (_e != hipSuccess) { free_regs(T); return hip_fail(_e); }                   \
    } while (0)
#define MAXK_SCAN(IN, OUT, COUNT)                                                                                              \
    do {                                                                                                                      \
        size_t _n = 0;                                                                                                        \
        MAXK_TRY_CLEAN(rocprim::exclusive_scan(nullptr, _n, IN, OUT, 0u, (size_t)(COUNT), rocprim::plus<uint32_t>(), s));      \
        char* _tmp;                                                                                                           \
        MAXK_TRY_CLEAN(get(_tmp, (int64_t)_n));                                                                               \
        MAXK_TRY_CLEAN(rocprim::exclusive_scan(_tmp, _n, IN, OUT, 0u, (size_t)(COUNT), rocprim::plus<uint32_t>(), s));         \
        MAXK_TRY_CLEAN(hipStreamSynchronize(s));                                                                              \
        drop(_tmp);                                                                                                           \
    } while (0)
    const auto blocks = [](int64_t n) { return dim3((unsigned)((n + 255) / 256)); };
    const dim3 wide((unsigned)std::min<int64_t>((nnz + 255) / 256, 65536));

    // shares of the destinations by falling degree, and their places
    if (shape.cap < 1) return MAXK_UNSUPPORTED;
    uint32_t *d_shares, *d_share0, *d_count1, *d_extra0;
    uint2* d_several;
    const int64_t most_several = nnz / shape.cap + 1;
    MAXK_TRY_CLEAN(get(d_shares, N + 1));
    MAXK_TRY_CLEAN(get(d_share0, N + 1));
    MAXK_TRY_CLEAN(get(d_count1, 1));
    MAXK_TRY_CLEAN(get(d_extra0, N));
    MAXK_TRY_CLEAN(get(d_several, most_several));
    MAXK_TRY_CLEAN(hipMemsetAsync(d_count1, 0, sizeof(uint32_t), s));
    hipLaunchKernelGGL(regs_shares_kernel, blocks(N + 1), dim3(256), 0, s, d_csc_ptr, N, shape.cap, d_shares, d_count1, d_several);
    MAXK_TRY_CLEAN(hipGetLastError());
    MAXK_SCAN(d_shares, d_share0, N + 1);
    uint32_t n_several = 0, n_shares32 = 0;
    MAXK_TRY_CLEAN(hipMemcpy(&n_several, d_count1, sizeof(uint32_t), hipMemcpyDeviceToHost));
    MAXK_TRY_CLEAN(hipMemcpy(&n_shares32, d_share0 + N, sizeof(uint32_t), hipMemcpyDeviceToHost));
    const int64_t n_shares = n_shares32;
    if (n_shares + N > 0x7FFFFFF0ll || shape.head > n_shares) return MAXK_UNSUPPORTED;
    if (n_several) {
        std::vector<uint2> several(n_several);
        MAXK_TRY_CLEAN(hipMemcpy(several.data(), d_several, sizeof(uint2) * several.size(), hipMemcpyDeviceToHost));
        std::sort(several.begin(), several.end(), [](const uint2& a, const uint2& b) { return a.x < b.x; });
        std::vector<RegsSplit> split;
        int32_t rows = 0;
        for (const uint2& x : several) {
            split.push_back(RegsSplit{(int32_t)x.x, rows, rows + (int32_t)x.y});
            rows += (int32_t)x.y;
        }
        T.n_split = (int64_t)split.size();
        T.extra_floats = (int64_t)rows * (kWave / shape.groups * shape.kr);
        MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_extra, sizeof(float) * (size_t)T.extra_floats));
        MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_split, sizeof(RegsSplit) * split.size()));
        MAXK_TRY_CLEAN(hipMemcpy(T.d_split, split.data(), sizeof(RegsSplit) * split.size(), hipMemcpyHostToDevice));
        hipLaunchKernelGGL(regs_extra_kernel, blocks(T.n_split), dim3(256), 0, s, T.d_split, T.n_split, d_extra0);
    }
    T.n_tail = n_shares - shape.head;
    uint32_t *d_degree, *d_degree_sorted, *d_place;
    int32_t *d_ids, *d_order;
    int2* d_goes;
    MAXK_TRY_CLEAN(get(d_degree, n_shares));
    MAXK_TRY_CLEAN(get(d_degree_sorted, n_shares));
    MAXK_TRY_CLEAN(get(d_ids, n_shares));
    MAXK_TRY_CLEAN(get(d_order, n_shares));
    MAXK_TRY_CLEAN(get(d_place, n_shares));
    MAXK_TRY_CLEAN(get(d_goes, n_shares));
    hipLaunchKernelGGL(regs_share_kernel, blocks(N), dim3(256), 0, s, d_csc_ptr, d_share0, N, d_extra0, d_degree, d_ids, d_goes);
    {
        size_t n = 0;
        char* tmp;
        MAXK_TRY_CLEAN(rocprim::radix_sort_pairs_desc(nullptr, n, d_degree, d_degree_sorted, d_ids, d_order, (size_t)n_shares, 0, 32, s));
        MAXK_TRY_CLEAN(get(tmp, (int64_t)n));
        MAXK_TRY_CLEAN(rocprim::radix_sort_pairs_desc(tmp, n, d_degree, d_degree_sorted, d_ids, d_order, (size_t)n_shares, 0, 32, s));
        MAXK_TRY_CLEAN(hipStreamSynchronize(s));
        drop(tmp);
    }
    MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_node, sizeof(int32_t) * (size_t)(per_set * S)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_row, sizeof(int32_t) * (size_t)(per_set * S)));
    MAXK_TRY_CLEAN(hipMemsetAsync(T.d_node, 0xFF, sizeof(int32_t) * (size_t)(per_set * S), s));
    MAXK_TRY_CLEAN(hipMemsetAsync(T.d_row, 0xFF, sizeof(int32_t) * (size_t)(per_set * S), s));
    uint32_t* d_entries;
    MAXK_TRY_CLEAN(get(d_entries, per_set * S));
    hipLaunchKernelGGL(regs_place_kernel, blocks(n_shares), dim3(256), 0, s, d_order, d_goes, n_shares, shape.head, shape.spread, shape.groups, slots,
                       shape.kr, d_degree_sorted, d_place, T.d_node, T.d_row, d_entries);
    MAXK_TRY_CLEAN(hipGetLastError());

    // The order that a set takes its rows in.  By degree: sources with most entries first, so that the sets that run at a time
    // bring the same rows (2.4 M nodes, k = 64: 6.4 against 6.9 ms); even sets do so in any order, and with the sources as they
    // come every step has about the same entries (115 M entries, k = 32: 2.42 against 2.70 ms).
    int32_t *d_src_order, *d_rank;
    uint32_t* d_src_degree;
    MAXK_TRY_CLEAN(get(d_src_degree, N));
    MAXK_TRY_CLEAN(get(d_src_order, N));
    MAXK_TRY_CLEAN(get(d_rank, N));
    hipLaunchKernelGGL(regs_degree_kernel, blocks(N), dim3(256), 0, s, d_rowptr, N, d_degree, d_ids);
    if (shape.ranges) {
        MAXK_TRY_CLEAN(hipMemcpyAsync(d_src_order, d_ids, sizeof(int32_t) * (size_t)N, hipMemcpyDeviceToDevice, s));
    } else {
        size_t n = 0;
        char* tmp;
        MAXK_TRY_CLEAN(rocprim::radix_sort_pairs_desc(nullptr, n, d_degree, d_src_degree, d_ids, d_src_order, (size_t)N, 0, 32, s));
        MAXK_TRY_CLEAN(get(tmp, (int64_t)n));
        MAXK_TRY_CLEAN(rocprim::radix_sort_pairs_desc(tmp, n, d_degree, d_src_degree, d_ids, d_src_order, (size_t)N, 0, 32, s));
        MAXK_TRY_CLEAN(hipStreamSynchronize(s));
        drop(tmp);
    }
    hipLaunchKernelGGL(regs_rank_kernel, blocks(N), dim3(256), 0, s, d_src_order, N, d_rank);

    // the rows that each set uses
    uint32_t *d_where, *d_used, *d_count, *d_before;
    MAXK_TRY_CLEAN(get(d_where, nnz));
    MAXK_TRY_CLEAN(get(d_used, n_words));
    MAXK_TRY_CLEAN(get(d_count, n_words + 1));
    MAXK_TRY_CLEAN(get(d_before, n_words + 1));
    MAXK_TRY_CLEAN(hipMemsetAsync(d_used, 0, sizeof(uint32_t) * (size_t)n_words, s));
    hipLaunchKernelGGL(regs_mark_kernel, wide, dim3(256), 0, s, d_csc_ptr, d_csc_src, N, nnz, d_share0, d_place, d_rank, words, d_where, d_used);
    hipLaunchKernelGGL(regs_popcount_kernel, blocks(n_words + 1), dim3(256), 0, s, d_used, n_words, d_count);
    MAXK_TRY_CLEAN(hipGetLastError());
    MAXK_SCAN(d_count, d_before, n_words + 1);
    drop(d_count);
    drop(d_degree);
    drop(d_ids);
    drop(d_order);
    drop(d_place);
    std::vector<uint32_t> row0((size_t)S + 1), tile0((size_t)S + 1);
    MAXK_TRY_CLEAN(hipMemcpy2D(row0.data(), sizeof(uint32_t), d_before, sizeof(uint32_t) * (size_t)words, sizeof(uint32_t), (size_t)S + 1,
                               hipMemcpyDeviceToHost));
    for (int32_t i = 0; i < S; ++i) tile0[(size_t)i + 1] = tile0[(size_t)i] + (row0[(size_t)i + 1] - row0[(size_t)i] + (uint32_t)tile_rows - 1) / (uint32_t)tile_rows;
    const int64_t n_tiles = tile0[(size_t)S], n_lists = n_tiles * kRegsWaves * shape.groups;
    if (n_lists >= (int64_t)1 << 31) { free_regs(T); return MAXK_UNSUPPORTED; }
    uint32_t *d_rows, *d_tile0;
    MAXK_TRY_CLEAN(get(d_rows, row0[(size_t)S]));
    MAXK_TRY_CLEAN(get(d_tile0, S + 1));
    MAXK_TRY_CLEAN(hipMemcpy(d_tile0, tile0.data(), sizeof(uint32_t) * ((size_t)S + 1), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(regs_rows_kernel, blocks(n_words), dim3(256), 0, s, d_used, d_before, n_words, words, d_src_order, d_rows);
    const RegsTables t = {d_used, d_before, d_tile0, d_rank, words, tile_rows, shape.pitch, shape.groups, shape.kr};

    // entries by list
    uint32_t *d_key, *d_key_sorted, *d_start;
    uint2 *d_entry, *d_entry_sorted;
    MAXK_TRY_CLEAN(get(d_key, nnz));
    MAXK_TRY_CLEAN(get(d_entry, nnz));
    hipLaunchKernelGGL(regs_keys_kernel, wide, dim3(256), 0, s, t, d_csc_src, d_csc_val, d_where, nnz, (uint32_t)n_lists, d_key, d_entry);
    MAXK_TRY_CLEAN(hipGetLastError());
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
    drop(d_where);
    MAXK_TRY_CLEAN(get(d_key_sorted, nnz));
    MAXK_TRY_CLEAN(get(d_entry_sorted, nnz));
    {
        unsigned bits = 1;
        while (bits < 32 && ((int64_t)1 << bits) <= n_lists) ++bits;
        size_t n = 0;
        char* tmp;
        MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(nullptr, n, d_key, d_key_sorted, d_entry, d_entry_sorted, (size_t)nnz, 0, bits, s));
        MAXK_TRY_CLEAN(get(tmp, (int64_t)n));
        MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(tmp, n, d_key, d_key_sorted, d_entry, d_entry_sorted, (size_t)nnz, 0, bits, s));
        MAXK_TRY_CLEAN(hipStreamSynchronize(s));
        drop(tmp);
    }
    drop(d_key);
    drop(d_entry);
    MAXK_TRY_CLEAN(get(d_start, n_lists + 1));
    hipLaunchKernelGGL(regs_starts_kernel, blocks(n_lists + 1), dim3(256), 0, s, d_key_sorted, nnz, n_lists, d_start);

    // steps, records and headers
    uint32_t *d_steps, *d_step0, *d_records, *d_record0;
    uint8_t* d_cost;
    uint32_t* d_pos;
    MAXK_TRY_CLEAN(get(d_steps, n_tiles + 1));
    MAXK_TRY_CLEAN(get(d_step0, n_tiles + 1));
    MAXK_TRY_CLEAN(get(d_records, n_tiles * kRegsWaves + 1));
    MAXK_TRY_CLEAN(get(d_record0, n_tiles * kRegsWaves + 1));
    hipLaunchKernelGGL(regs_tiles_kernel, blocks(n_tiles + 1), dim3(256), 0, s, t, d_start, n_tiles, d_steps, d_records);
    MAXK_TRY_CLEAN(hipGetLastError());
    MAXK_SCAN(d_steps, d_step0, n_tiles + 1);
    MAXK_SCAN(d_records, d_record0, n_tiles * kRegsWaves + 1);
    uint32_t n_steps = 0, n_records = 0, n_entries = 0;
    MAXK_TRY_CLEAN(hipMemcpy(&n_steps, d_step0 + n_tiles, sizeof(uint32_t), hipMemcpyDeviceToHost));
    MAXK_TRY_CLEAN(hipMemcpy(&n_records, d_record0 + n_tiles * kRegsWaves, sizeof(uint32_t), hipMemcpyDeviceToHost));
    MAXK_TRY_CLEAN(hipMemcpy(&n_entries, d_start + n_lists, sizeof(uint32_t), hipMemcpyDeviceToHost));
    // the sums are of 32 bits: refuse what could have wrapped (a list ends with less than a batch of padding, a record has an entry)
    const int64_t batch = regs_batch_records(shape.groups, shape.kr);
    if ((int64_t)n_entries * (shape.groups > 2 ? 2 : 1) + n_tiles * kRegsWaves * batch >= (int64_t)0xFFFF0000 || n_steps > 0x3FFFFFFFu) {
        free_regs(T);
        return MAXK_UNSUPPORTED;
    }
    // the kernel reads headers past its last step, and their lists: empty ones, at record 0 like every empty list
    const int64_t all_steps = (int64_t)n_steps + kRegsSpareSteps, all_records = std::max<int64_t>(n_records, 1);
    MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_hdr, sizeof(uint32_t) * (size_t)(all_steps * kRegsWaves * layout.head)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_rec, sizeof(uint4) * (size_t)all_records));
    MAXK_TRY_CLEAN(get(d_cost, n_steps));
    MAXK_TRY_CLEAN(get(d_pos, n_steps));
    MAXK_TRY_CLEAN(hipMemsetAsync(T.d_hdr, 0, sizeof(uint32_t) * (size_t)(all_steps * kRegsWaves * layout.head), s));
    hipLaunchKernelGGL(regs_padding_kernel, wide, dim3(256), 0, s, T.d_rec, all_records, (uint32_t)(slots * shape.kr));
    hipLaunchKernelGGL(regs_headers_kernel, blocks((n_tiles + kRegsSpareSteps) * kRegsWaves), dim3(256), 0, s, t, d_start, d_rows, n_tiles, S, layout.rows,
                           layout.head, d_step0, d_record0, T.d_hdr, d_cost, d_pos);
    hipLaunchKernelGGL(regs_records_kernel, wide, dim3(256), 0, s, t, d_key_sorted, d_entry_sorted, (int64_t)n_entries, d_start, d_record0,
                       reinterpret_cast<uint2*>(T.d_rec));
    MAXK_TRY_CLEAN(hipGetLastError());
    std::vector<uint32_t> step0((size_t)n_tiles + 1);
    std::vector<uint8_t> cost((size_t)std::max<uint32_t>(n_steps, 1));
    MAXK_TRY_CLEAN(hipMemcpy(step0.data(), d_step0, sizeof(uint32_t) * step0.size(), hipMemcpyDeviceToHost));
    std::vector<uint32_t> pos(cost.size());
    MAXK_TRY_CLEAN(hipMemcpy(pos.data(), d_pos, sizeof(uint32_t) * n_steps, hipMemcpyDeviceToHost));
    MAXK_TRY_CLEAN(hipMemcpy(cost.data(), d_cost, n_steps, hipMemcpyDeviceToHost));
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));

    // Units: a set's steps, cut by what they cost.  Parts: a unit's steps, cut where the sums of a destination get long: a
    // set's mean in-entries (seen from an entry) over `run` times, at most kRegsMaxParts; the first slots by themselves, oftener.
    // That is a mean: a hub has more entries than its set's, and they may crowd into few of the steps.  So no sum may take more
    // than `longest` either: the entries of every sum that could are counted, and a set where one does is cut more often.  (126 M
    // entries on 2.4 M nodes, k = 64, the eight destinations of up to 156 k in-entries: error against 64 bits 8.5e-7 by the mean alone,
    // some 1,900 entries a sum, 2.9e-7 so, pull 4.9e-7; 6.67 / 6.62 ms, 5 ms more to build.)
    std::vector<uint32_t> degree((size_t)shape.head);
    MAXK_TRY_CLEAN(hipMemcpy(degree.data(), d_degree_sorted, sizeof(uint32_t) * degree.size(), hipMemcpyDeviceToHost));
    std::vector<RegsUnit> units;
    std::vector<RegsSum> sums;
    std::vector<RegsPart> part_end;
    std::vector<int2> part_range((size_t)S);
    struct Parts { double least[2] = {}, have[2] = {}; };  // of the first slots and of the others: asked for by `longest`; cut
    std::vector<Parts> parts_of((size_t)S);
    const auto step_cost = [&](uint32_t st) { return std::max(14.0, 8.0 + (double)cost[st]); };
    double total = 0.0;
    for (uint32_t st = 0; st < n_steps; ++st) total += step_cost(st);
    const double share = total / (256.0 * std::clamp(std::round(total / (256.0 * kRegsUnitCost)), 1.0, 4.0)) + 1.0;
    const int64_t whole_floats = (int64_t)kRegsWaves * slots * shape.kr * kWave, hot_floats = (int64_t)kRegsWaves * kRegsHotSlots * shape.kr * kWave;
    const int64_t per_run = per_set * shape.spread, hot_per_run = per_run / slots * kRegsHotSlots;
    const auto cut = [&] {
        units.clear();
        sums.clear();
        part_end.clear();
        for (int32_t set = 0; set < S; ++set) {
            const uint32_t b = step0[tile0[(size_t)set]], e = step0[tile0[(size_t)set + 1]];
            Parts& of = parts_of[(size_t)set];
            double all = 0.0, entries[2] = {}, squares[2] = {};  // of the first slots and of the others
            for (uint32_t st = b; st < e; ++st) all += step_cost(st);
            const int64_t run0 = set / shape.spread * per_run, run1 = std::min<int64_t>(run0 + per_run, shape.head);
            for (int64_t q = run0; q < run1; q += shape.spread) {
                const int cold = q - run0 >= hot_per_run;
                entries[cold] += degree[(size_t)q];
                squares[cold] += (double)degree[(size_t)q] * degree[(size_t)q];
            }
            const int pieces = shape.ranges ? shape.ranges : std::max(1, (int)(all / share + 0.5));
            const auto wanted = [&](int cold) {
                const double mean = shape.run && entries[cold] > 0.0 ? std::min(kRegsMaxParts[cold], squares[cold] / entries[cold] / shape.run) : 1.0;
                const int64_t first = run0 + (cold ? hot_per_run : 0);
                if (shape.longest && first < run1) of.least[cold] = std::max(of.least[cold], (double)degree[(size_t)first] / shape.longest);
                return std::max(mean, std::min(of.least[cold], 4.0 * (e - b)));
            };
            const auto times = [](double a, int b) { return std::max(1, (int)std::ceil(a / b)); };
            const int whole = times(wanted(1), pieces), per_unit = whole * times(wanted(0), pieces * whole), parts = pieces * per_unit;
            of.have[0] = parts;
            of.have[1] = pieces * whole;
            const int32_t first_part = (int32_t)part_end.size();
            uint32_t at = b;
            double sum = 0.0;
            for (int i = 0; i < pieces; ++i) {
                RegsUnit u = {set, (int32_t)at, 0, (int32_t)part_end.size(), 0};
                for (int j = 0; j < per_unit; ++j) {
                    const int cut = i * per_unit + j + 1;
                    const uint32_t from = at;
                    while (at < e && (cut == parts || sum < all * cut / parts)) sum += step_cost(at++);
                    const int leave = (j + 1) % (per_unit / whole) == 0 ? slots : kRegsHotSlots;
                    if (parts > 1 && at > from) part_end.push_back(RegsPart{(int32_t)at, leave, 0});
                    else if ((int32_t)part_end.size() > u.part_begin) part_end.back().slots = std::max(part_end.back().slots, leave);  // (fewer steps than parts)
                }
                u.end = (int32_t)at;
                u.part_end = (int32_t)part_end.size();
                if (u.begin < u.end || parts == 1) units.push_back(u);
            }
            part_range[(size_t)set] = make_int2(first_part, (int32_t)part_end.size());
            if (parts > 1) sums.push_back(RegsSum{set, first_part, (int32_t)part_end.size(), 0, 0});
        }
        // parts in which all slots leave first, set after set, then the others
        int64_t n_whole = 0, n_hot = 0;
        for (const RegsPart& x : part_end) (x.slots == slots ? n_whole : n_hot) += 1;
        T.hot_parts = n_whole * whole_floats;
        T.part_floats = T.hot_parts + n_hot * hot_floats;
        int32_t whole = 0, hot = 0;
        for (RegsSum& x : sums) {
            const int32_t b = x.whole_begin, e = x.whole_end;
            x.whole_begin = whole;
            x.hot_begin = hot;
            for (int32_t i = b; i < e; ++i) {
                RegsPart& q = part_end[(size_t)i];
                q.at = q.slots == slots ? whole++ * whole_floats : T.hot_parts + hot++ * hot_floats;
            }
            x.whole_end = whole;
            x.hot_end = hot;
        }
    };
    const bool limited = shape.longest && !degree.empty() && degree[0] > (uint32_t)shape.longest;
    int2* d_part_range;
    uint32_t* d_most;
    MAXK_TRY_CLEAN(get(d_part_range, S));
    MAXK_TRY_CLEAN(get(d_most, 2 * S));
    int64_t first_floats = 0;
    for (int tries = 0;; ++tries) {
        cut();
        if (tries == 0) first_floats = T.part_floats;
        if (!sums.empty()) {
            (void)hipFree(T.d_part);
            (void)hipFree(T.d_parts);
            T.d_part = nullptr;
            T.d_parts = nullptr;
            MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_part, sizeof(RegsPart) * std::max<size_t>(part_end.size(), 1)));
            MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_parts, sizeof(float) * (size_t)std::max<int64_t>(T.part_floats, 1)));
            MAXK_TRY_CLEAN(hipMemcpy(T.d_part, part_end.data(), sizeof(RegsPart) * part_end.size(), hipMemcpyHostToDevice));
        }
        if (!limited || part_end.empty()) break;
        uint32_t* const count = reinterpret_cast<uint32_t*>(T.d_parts);
        std::vector<uint32_t> most(2 * (size_t)S);
        MAXK_TRY_CLEAN(hipMemcpy(d_part_range, part_range.data(), sizeof(int2) * part_range.size(), hipMemcpyHostToDevice));
        MAXK_TRY_CLEAN(hipMemsetAsync(count, 0, sizeof(uint32_t) * (size_t)T.part_floats, s));
        MAXK_TRY_CLEAN(hipMemsetAsync(d_most, 0, sizeof(uint32_t) * most.size(), s));
        hipLaunchKernelGGL(regs_longest_kernel, wide, dim3(256), 0, s, t, d_key_sorted, d_entry_sorted, (int64_t)n_entries, d_start, d_step0, S, slots,
                           d_entries, d_part_range, T.d_part, (uint32_t)shape.longest, count, d_most);
        MAXK_TRY_CLEAN(hipGetLastError());
        MAXK_TRY_CLEAN(hipMemcpy(most.data(), d_most, sizeof(uint32_t) * most.size(), hipMemcpyDeviceToHost));
        bool good = true;
        for (int32_t set = 0; set < S; ++set)
            for (int c = 0; c < 2; ++c)
                if (const uint32_t n = most[2 * (size_t)set + (size_t)c]; n) {
                    parts_of[(size_t)set].least[c] = parts_of[(size_t)set].have[c] * std::max(1.25, 1.1 * n / shape.longest);
                    good = false;
                }
        if (good) break;
        // a graph whose order needs far more parts than were reckoned with is for the other kernels
        if (tries == 8 || T.part_floats > 2 * first_floats + 64000000) {
            free_regs(T);
            return MAXK_UNSUPPORTED;
        }
    }
    // 256 units run at a time, unit u on XCD u % 8: an XCD gets units that begin with about the same rows
    std::vector<RegsUnit> placed(units.size());
    for (size_t c = 0; c < units.size(); c += 256) {
        const size_t n = std::min<size_t>(256, units.size() - c);
        const auto begins = [&](const RegsUnit& u) { return u.begin < u.end ? pos[(size_t)u.begin] : 0xFFFFFFFFu; };
        std::stable_sort(units.begin() + (int64_t)c, units.begin() + (int64_t)(c + n), [&](const RegsUnit& x, const RegsUnit& y) { return begins(x) < begins(y); });
        size_t from = 0;
        for (size_t x = 0; x < 8; ++x)
            for (size_t m = x; m < n; m += 8) placed[c + m] = units[c + from++];
    }
    units.swap(placed);
    MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_unit, sizeof(RegsUnit) * units.size()));
    MAXK_TRY_CLEAN(hipMemcpy(T.d_unit, units.data(), sizeof(RegsUnit) * units.size(), hipMemcpyHostToDevice));
    if (!sums.empty()) {
        MAXK_TRY_CLEAN(hipMalloc((void**)&T.d_sum, sizeof(RegsSum) * sums.size()));
        MAXK_TRY_CLEAN(hipMemcpy(T.d_sum, sums.data(), sizeof(RegsSum) * sums.size(), hipMemcpyHostToDevice));
    }
#undef MAXK_TRY_CLEAN
#undef MAXK_SCAN
    T.shape = shape;
    T.n_units = (int64_t)units.size();
    T.n_sums = (int64_t)sums.size();
    T.n_steps = n_steps;
    T.n_records = n_records;
    T.n_parts = (int64_t)part_end.size();
    return MAXK_OK;
}

namespace {

// Adds up the parts of a set; a thread four positions.  Bound by the read of the parts, each wanted once: 16-byte loads, eight under
// way (one conditional load of 4 bytes after the other took 0.46 ms for 1.3 GB, 115 M entries, k = 64).
__global__ __launch_bounds__(256) void regs_sum_kernel(const RegsSum* __restrict__ sum, const int32_t* __restrict__ to, const float* __restrict__ parts,
                                                       int64_t hot_parts, int32_t slots, int32_t groups, int32_t kr, int64_t N, int32_t k,
                                                       float* __restrict__ dXs, float* __restrict__ extra)
{
    const int per_wave = slots * kr, hot_per_wave = kRegsHotSlots * kr, rows = kRegsWaves * per_wave, blocks = (rows + 15) / 16;
    const RegsSum u = sum[blockIdx.x / blocks];
    const int row = (int)(blockIdx.x % blocks) * 16 + (int)threadIdx.x / 16, lane = (int)threadIdx.x % 16 * 4;  // accumulator; first lane
    if (row >= rows) return;
    const int w = row / per_wave, r = row % per_wave, width = kWave / groups;
    const int j = to[((int64_t)u.set * kRegsWaves + w) * (slots * groups) + r / kr * groups + lane / width], p = lane % width + r % kr * kWave;
    double x[4] = {0.0, 0.0, 0.0, 0.0};
    const auto add = [&](const float* __restrict__ at, int64_t stride, int n) {
        int i = 0;
        for (; i + 8 <= n; i += 8) {
            float4 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = load_once(reinterpret_cast<const float4*>(at + (i + q) * stride));
#pragma unroll
            for (int q = 0; q < 8; ++q) { x[0] += v[q].x; x[1] += v[q].y; x[2] += v[q].z; x[3] += v[q].w; }
        }
#pragma unroll 4
        for (; i < n; ++i) {
            const float4 v = load_once(reinterpret_cast<const float4*>(at + i * stride));
            x[0] += v.x; x[1] += v.y; x[2] += v.z; x[3] += v.w;
        }
    };
    const int64_t whole = (int64_t)rows * kWave, hot = (int64_t)kRegsWaves * hot_per_wave * kWave;
    add(parts + u.whole_begin * whole + (int64_t)row * kWave + lane, whole, u.whole_end - u.whole_begin);
    if (r < hot_per_wave)
        add(parts + hot_parts + u.hot_begin * hot + ((int64_t)w * hot_per_wave + r) * kWave + lane, hot, u.hot_end - u.hot_begin);
    if (j < 0) return;
    float* const out = (j < N ? dXs : extra - N * k) + ((int64_t)j * k + p);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (p + i < k) out[i] = (float)x[i];
}

// Adds up the shares of the destinations that are several ones
__global__ __launch_bounds__(128) void regs_split_kernel(const RegsSplit* __restrict__ split, const float* __restrict__ extra, int32_t k,
                                                         float* __restrict__ dXs)
{
    const RegsSplit u = split[blockIdx.x];
    const int p = threadIdx.x;
    if (p >= k) return;
    double x = 0.0;
#pragma unroll 4
    for (int i = u.row_begin; i < u.row_end; ++i) x += (double)extra[(int64_t)i * k + p];
    dXs[(int64_t)u.node * k + p] = (float)x;
}

}  // namespace

maxk_status launch_bwd_regs(const RegsSet& T, const void* dY, int value_type, const void* sp_index, int index_bytes, int64_t N, int dim,
                            int k, float* dXs, hipStream_t s)
{
    RegsShape sh;
    if (!aligned(dY, 16) || !regs_fits(dim, value_bytes(value_type), k, sh) || sh.pitch != T.shape.pitch || sh.groups != T.shape.groups ||
        sh.kr != T.shape.kr)
        return MAXK_UNSUPPORTED;
    const maxk_status st = value_type == MAXK_VALUE_BF16 ? launch_regs_format<MAXK_VALUE_BF16>(T, dY, sp_index, index_bytes, N, dim, k, dXs, s)
                           : value_type == MAXK_VALUE_F16 ? launch_regs_format<MAXK_VALUE_F16>(T, dY, sp_index, index_bytes, N, dim, k, dXs, s)
                                                          : launch_regs_format<MAXK_VALUE_F32>(T, dY, sp_index, index_bytes, N, dim, k, dXs, s);
    if (st != MAXK_OK) return st;
    if (T.n_sums) {
        const int32_t slots = regs_slots(sh.kr);
        hipLaunchKernelGGL(regs_sum_kernel, dim3((unsigned)((kRegsWaves * slots * sh.kr + 15) / 16 * T.n_sums)), dim3(256), 0, s, T.d_sum, T.d_row,
                           T.d_parts, T.hot_parts, slots, sh.groups, sh.kr, N, k, dXs, T.d_extra);
        MAXK_LAUNCH_CHECK();
    }
    if (T.n_split) {
        hipLaunchKernelGGL(regs_split_kernel, dim3((unsigned)T.n_split), dim3(128), 0, s, T.d_split, T.d_extra, k, dXs);
        MAXK_LAUNCH_CHECK();
    }
    return MAXK_OK;
}

}  // namespace maxk
