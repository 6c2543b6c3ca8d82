// Graph handle: load-time preprocessing of the adjacency (the paper's O(n)
// partition of rows into edge groups "during graph loading", Sec. 4.1 / 4.2),
// and the extern "C" entry points of the library.
//
// Preprocessing builds, once per graph:
//   - the forward work-item list: rows cut into runs of at most `chunk` stored
//     entries, ordered longest first so the heavy tail of a power-law degree
//     distribution starts early and the short rows fill in behind it;
//   - A^T as value-carrying CSC (stable radix sort of the entries by column, so
//     in-entries of a node stay ordered by source row: deterministic sums) and
//     its work-item list, for the pull backward kernel;
//   - one partial-sum workspace shared by all kernels of the handle.
#include <algorithm>
#include <bit>
#include <array>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <new>
#include <utility>
#include <vector>

#include <rocprim/rocprim.hpp>

#include "common.hpp"

struct maxk_graph {
    int64_t N = 0, nnz = 0;
    const int32_t* d_rowptr = nullptr;  // caller's CSR, aliased
    const int32_t* d_col = nullptr;
    const float* d_val = nullptr;
    maxk::ItemList csr_items;  // over rows of A
    std::vector<std::pair<int32_t, int64_t>> csr_lengths;  // entries of a work item of csr_items, how many such items; longest first
    maxk::ItemList csc_items;  // over columns of A (rows of A^T)
    int32_t* d_csc_ptr = nullptr;
    int32_t* d_csc_src = nullptr;
    float* d_csc_val = nullptr;
    uint32_t* d_csc_entry = nullptr;  // CSR entry id of every CSC position (the transposing permutation)
    float* d_partials = nullptr;
    int64_t partial_floats = 0;
    float* d_expand = nullptr;  // per-entry contributions of the expand/reduce backward kernel (nnz * k floats)
    int64_t expand_floats = 0;
    std::vector<maxk::SlabSet*> slab_cache;    // A^T regrouped per slab height (one per height ever asked for)
    std::vector<maxk::TiledSet*> tiled_cache;  // visit lists of the LDS-tiled kernel, one per (set size, k / 4)
    std::vector<maxk::RegsSet*> regs_cache;    // A^T regrouped for the register-tiled kernel, one per shape
    struct RegsChoice { int32_t dim, val_bytes, k; maxk::RegsShape shape; };
    std::vector<RegsChoice> regs_choices;      // what regs_choice found, per shape
    std::vector<maxk::RegsShape> regs_refused; // tables that could not be built (see is_refused)
    int32_t bwd_regs = 0;
    std::vector<std::pair<int32_t, int64_t>> in_degrees;  // in-entries of a node, how many such nodes; most first
    std::vector<maxk::SweepSet*> sweep_cache;  // A regrouped for the forward sweep, one per (lane groups, rows of a bin)
    char* d_sliced = nullptr;   // slice-major copy of dY for the column-sliced pull (rows that are not whole cache lines)
    int64_t sliced_bytes = 0;
    std::vector<char*> sliced_before;  // smaller ones: a captured backward pass may still hold their address
    int64_t sliced_before_bytes = 0;
    char* d_packed = nullptr;   // forward kernel's per-call repack of a small-k CBSR (one record per node)
    int64_t packed_bytes = 0;
    int64_t max_degree = 0;      // longest row of A (entries with one source)
    int64_t max_in_degree = 0;   // longest column (entries with one destination)
    float hot_share[33] = {};    // share of the entries whose source is among the 2^i sources with most entries
    int32_t bwd_mode = MAXK_BWD_AUTO;
    int32_t chunk = 0;         // tuning knobs, read from the environment once, by maxk_graph_create
    int32_t slab_kb = 0;
    int32_t fwd_pack_max = 0;
    int32_t pull_form = 0;
    int32_t fwd_sweep = 0;
    std::vector<std::pair<int32_t, int32_t>> reserved;  // (dim, k) of maxk_graph_reserve*, none within another
    std::vector<std::array<int64_t, 4>> refused;  // tables that could not be built: {kind, shape}; a reserve tries them again
    int64_t test_alloc_limit = -1;  // test hook: tables and buffers of more bytes are refused (-1: none)
    int64_t test_denied = 0;        // how many were
    unsigned char* d_noalloc_scratch = nullptr;  // this device's copy of the library's fixed scratch array
    int device = 0;
};

// Scratch memory of maxk_spgemm_fwd_noalloc: a fixed array in the library's device image, one copy per GPU, alive
// until the process ends.  In host code this name is a handle for hipGetSymbolAddress only, never a pointer.
static __device__ __align__(256) unsigned char maxk_noalloc_scratch[MAXK_NOALLOC_SCRATCH_BYTES];

namespace maxk {

thread_local int32_t g_last_hip_error = 0;

namespace {

// Device address of the scratch array on the current device (asked for once per handle, by maxk_graph_create).
maxk_status noalloc_scratch_address(unsigned char** out)
{
    void* p = nullptr;
    MAXK_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(maxk_noalloc_scratch)));
    *out = static_cast<unsigned char*>(p);
    return p ? MAXK_OK : MAXK_HIP_ERROR;
}

int env_int(const char* name, int dflt, int lo, int hi)
{
    const char* v = std::getenv(name);
    if (!v || !*v) return dflt;
    long x = std::strtol(v, nullptr, 10);
    if (x < lo || x > hi) return dflt;
    return (int)x;
}

// Entries per work item when the caller sets none.  One wavefront walks an item serially, so a launch takes at least
// as long as its longest item: on a graph of a few million entries an item of 2048 outlasted all the other work.  A
// 4096th of the entries per item keeps that tail below the rest (MI355X, us at 2048 -> at this rule: 2.5 M entries,
// 169 k nodes, k=32: forward 150 -> 97, pull 387 -> 228, expand/reduce 336 -> 281; 1.2 M entries, 40 k nodes, k=13:
// forward 74 -> 50, pull 114 -> 49; 2.1 M entries, 4 k nodes, k=16: forward 49 -> 34).  From 8 M entries up the tail
// is hidden and shorter items only add partial rows (43 M entries: forward 1405 us at 2048, 1491 at 512).  Below
// 128 an item costs more to start than to walk.  A row of more than `chunk` entries makes at most 2 * len / chunk
// items, so there are never more than 8192 partial rows from this rule while it is below 2048: 32 MiB at the widest
// row, which the fixed scratch array of maxk_spgemm_fwd_noalloc holds.
int default_chunk(int64_t nnz)
{
    return (int)std::min<int64_t>(2048, std::max<int64_t>(128, (nnz + 4095) / 4096));
}

// Host side of the partition: ptr[n+1] -> items (longest first) + split rows.
void build_items(const std::vector<int32_t>& ptr, int64_t n, int chunk, std::vector<WorkItem>& items,
                 std::vector<SplitRow>& split, int64_t& n_slots, int64_t& max_len)
{
    items.clear();
    split.clear();
    n_slots = 0;
    max_len = 0;
    items.reserve((size_t)n + 1024);
    for (int64_t i = 0; i < n; ++i) {
        const int32_t b = ptr[i], e = ptr[i + 1];
        const int64_t len = (int64_t)e - b;
        max_len = std::max(max_len, len);
        if (len <= chunk) {
            items.push_back(WorkItem{(int32_t)i, b, e, -1});
        } else {
            // equal-sized pieces, each at most `chunk`
            const int64_t pieces = (len + chunk - 1) / chunk;
            split.push_back(SplitRow{(int32_t)i, (int32_t)n_slots, (int32_t)pieces});
            for (int64_t s = 0; s < pieces; ++s) {
                const int32_t pb = (int32_t)(b + len * s / pieces), pe = (int32_t)(b + len * (s + 1) / pieces);
                items.push_back(WorkItem{(int32_t)i, pb, pe, (int32_t)(n_slots + s)});
            }
            n_slots += pieces;
        }
    }
    std::stable_sort(items.begin(), items.end(), [](const WorkItem& a, const WorkItem& b) {
        return (a.end - a.begin) > (b.end - b.begin);
    });
}

// How many rows have each number of entries, most entries first, from the work items, which are in that order (2.4 M rows: 85 to 123 ms
// with a sort of all rows' lengths instead).
void count_lengths(const std::vector<int32_t>& ptr, const std::vector<WorkItem>& items, const std::vector<SplitRow>& split,
                   std::vector<std::pair<int32_t, int64_t>>& out)
{
    const auto add = [&](int32_t length) {
        if (out.empty() || out.back().first != length) out.emplace_back(length, 0);
        ++out.back().second;
    };
    std::vector<int32_t> longer;  // than an item
    for (const SplitRow& r : split) longer.push_back(ptr[(size_t)r.row + 1] - ptr[(size_t)r.row]);
    std::sort(longer.begin(), longer.end(), std::greater<>());
    for (const int32_t length : longer) add(length);
    for (const WorkItem& w : items)
        if (w.slot < 0) add(w.end - w.begin);
}

maxk_status upload_items(const std::vector<WorkItem>& items, const std::vector<SplitRow>& split, int64_t n_slots,
                         ItemList& L, hipStream_t s)
{
    L.n_items = (int64_t)items.size();
    L.n_split = (int64_t)split.size();
    L.n_slots = n_slots;
    L.n_entries = 0;
    for (const WorkItem& w : items) L.n_entries += w.end - w.begin;
    L.n_long = std::partition_point(items.begin(), items.end(),
                                    [](const WorkItem& w) { return w.end - w.begin > kSlicedLongItem; }) - items.begin();
    if (L.n_items) {
        MAXK_HIP_TRY(hipMalloc((void**)&L.d_items, sizeof(WorkItem) * items.size()));
        MAXK_HIP_TRY(hipMemcpyAsync(L.d_items, items.data(), sizeof(WorkItem) * items.size(), hipMemcpyHostToDevice, s));
    }
    if (L.n_split) {
        MAXK_HIP_TRY(hipMalloc((void**)&L.d_split, sizeof(SplitRow) * split.size()));
        MAXK_HIP_TRY(hipMemcpyAsync(L.d_split, split.data(), sizeof(SplitRow) * split.size(), hipMemcpyHostToDevice, s));
    }
    MAXK_HIP_TRY(hipStreamSynchronize(s));  // the host vectors go out of scope after this
    return MAXK_OK;
}

// row_of[p] = the row that stored entry p belongs to (binary search in rowptr)
__global__ __launch_bounds__(256) void entry_rows_kernel(const int32_t* __restrict__ rowptr, int64_t N, int64_t nnz,
                                                         int32_t* __restrict__ row_of, uint32_t* __restrict__ iota)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += stride) {
        int64_t lo = 0, hi = N;  // largest i with rowptr[i] <= p
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)rowptr[mid] <= p) lo = mid; else hi = mid;
        }
        row_of[p] = (int32_t)lo;
        iota[p] = (uint32_t)p;
    }
}

// count[j] = stored entries in column j; ids outside [0,N) are tallied in count[N]
__global__ __launch_bounds__(256) void column_histogram_kernel(const int32_t* __restrict__ col, int64_t N,
                                                               int64_t nnz, int32_t* __restrict__ count)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += stride) {
        const int32_t c = col[p];
        atomicAdd(&count[(c >= 0 && (int64_t)c < N) ? c : N], 1);
    }
}

__global__ __launch_bounds__(256) void gather_transposed_kernel(const uint32_t* __restrict__ perm,
                                                                const int32_t* __restrict__ row_of,
                                                                const float* __restrict__ val, int64_t nnz,
                                                                int32_t* __restrict__ csc_src,
                                                                float* __restrict__ csc_val)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nnz; q += stride) {
        const uint32_t p = perm[q];
        csc_src[q] = row_of[p];
        csc_val[q] = val[p];
    }
}

// A^T in CSC: csc_ptr[N+1] (host copy returned), csc_src / csc_val on the device.
maxk_status build_csc(maxk_graph* g, std::vector<int32_t>& h_csc_ptr, hipStream_t s)
{
    const int64_t N = g->N, nnz = g->nnz;
    h_csc_ptr.assign((size_t)N + 1, 0);
    MAXK_HIP_TRY(hipMalloc((void**)&g->d_csc_ptr, sizeof(int32_t) * (size_t)(N + 1)));
    if (nnz == 0) {
        MAXK_HIP_TRY(hipMemsetAsync(g->d_csc_ptr, 0, sizeof(int32_t) * (size_t)(N + 1), s));
        MAXK_HIP_TRY(hipStreamSynchronize(s));
        return MAXK_OK;
    }
    MAXK_HIP_TRY(hipMalloc((void**)&g->d_csc_src, sizeof(int32_t) * (size_t)nnz));
    MAXK_HIP_TRY(hipMalloc((void**)&g->d_csc_val, sizeof(float) * (size_t)nnz));

    int32_t *d_row_of = nullptr, *d_count = nullptr;
    uint32_t *d_iota = nullptr, *d_keys_out = nullptr;
    MAXK_HIP_TRY(hipMalloc((void**)&g->d_csc_entry, sizeof(uint32_t) * (size_t)nnz));
    uint32_t* d_perm = g->d_csc_entry;  // kept: the reduce phase of the backward pass gathers through it
    void* d_tmp = nullptr;
    maxk_status st = MAXK_OK;
    auto cleanup = [&]() {
        (void)hipFree(d_row_of); (void)hipFree(d_count); (void)hipFree(d_iota);
        (void)hipFree(d_keys_out); (void)hipFree(d_tmp);
    };
#define MAXK_TRY_CLEAN(expr)                        \
    do {                                            \
        hipError_t _e = (expr);                     \
        if (_e != hipSuccess) { cleanup(); return hip_fail(_e); } \
    } while (0)
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_row_of, sizeof(int32_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_iota, sizeof(uint32_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_keys_out, sizeof(uint32_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_count, sizeof(int32_t) * (size_t)(N + 1)));
    MAXK_TRY_CLEAN(hipMemsetAsync(d_count, 0, sizeof(int32_t) * (size_t)(N + 1), s));

    const unsigned blocks = (unsigned)std::min<int64_t>((nnz + 255) / 256, 65536);
    hipLaunchKernelGGL(entry_rows_kernel, dim3(blocks), dim3(256), 0, s, g->d_rowptr, N, nnz, d_row_of, d_iota);
    hipLaunchKernelGGL(column_histogram_kernel, dim3(blocks), dim3(256), 0, s, g->d_col, N, nnz, d_count);
    MAXK_TRY_CLEAN(hipGetLastError());

    // stable sort of entry ids by column: in-entries of a node keep ascending source row
    int end_bit = 1;
    while (end_bit < 32 && ((int64_t)1 << end_bit) < N) ++end_bit;
    size_t tmp_bytes = 0;
    const uint32_t* keys_in = reinterpret_cast<const uint32_t*>(g->d_col);
    MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(nullptr, tmp_bytes, keys_in, d_keys_out, d_iota, d_perm, (size_t)nnz, 0,
                                             (unsigned)end_bit, s));
    MAXK_TRY_CLEAN(hipMalloc(&d_tmp, tmp_bytes ? tmp_bytes : 16));
    MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(d_tmp, tmp_bytes, keys_in, d_keys_out, d_iota, d_perm, (size_t)nnz, 0,
                                             (unsigned)end_bit, s));
    hipLaunchKernelGGL(gather_transposed_kernel, dim3(blocks), dim3(256), 0, s, d_perm, d_row_of, g->d_val, nnz,
                       g->d_csc_src, g->d_csc_val);
    MAXK_TRY_CLEAN(hipGetLastError());

    // column counts -> pointers (host scan over N values)
    std::vector<int32_t> h_count((size_t)N + 1);
    MAXK_TRY_CLEAN(hipMemcpyAsync(h_count.data(), d_count, sizeof(int32_t) * (size_t)(N + 1), hipMemcpyDeviceToHost, s));
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
    int64_t run = 0;
    for (int64_t j = 0; j < N; ++j) {
        h_csc_ptr[(size_t)j] = (int32_t)run;
        run += h_count[(size_t)j];
    }
    h_csc_ptr[(size_t)N] = (int32_t)run;
    if (run != nnz) st = MAXK_INVALID_ARGUMENT;  // a column id fell outside [0,N)
    MAXK_TRY_CLEAN(hipMemcpyAsync(g->d_csc_ptr, h_csc_ptr.data(), sizeof(int32_t) * (size_t)(N + 1), hipMemcpyHostToDevice, s));
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
#undef MAXK_TRY_CLEAN
    cleanup();
    return st;
}

// The test hook's stand-in for a device without room for `bytes` more
bool denied(maxk_graph* g, int64_t bytes)
{
    if (g->test_alloc_limit < 0 || bytes <= g->test_alloc_limit) return false;
    ++g->test_denied;
    return true;
}

// A table or buffer that could not be built is not asked for again by compute calls: each try synchronises the device
// and may allocate most of what it needs before it fails, and one that succeeds later would change the kernel mid-run.
using RefusedKey = std::array<int64_t, 4>;
enum : int64_t { kRefusedSweep, kRefusedSlab, kRefusedTiled, kRefusedExpand, kRefusedSliced };

bool is_refused(const maxk_graph* g, const RefusedKey& key)
{
    return std::find(g->refused.begin(), g->refused.end(), key) != g->refused.end();
}

void note_refused(maxk_graph* g, const RefusedKey& key)
{
    if (is_refused(g, key)) return;
    try {
        g->refused.push_back(key);
    } catch (const std::bad_alloc&) {  // then the next call tries again
    }
}

void forget_refused(maxk_graph* g, const RefusedKey& key) { std::erase(g->refused, key); }

maxk_status allocate(maxk_graph* g, void** out, int64_t bytes, const RefusedKey& key)
{
    const maxk_status st = denied(g, bytes) ? MAXK_OUT_OF_MEMORY : [&] {
        const hipError_t e = hipMalloc(out, (size_t)bytes);
        return e == hipSuccess ? MAXK_OK : hip_fail(e);
    }();
    if (st == MAXK_OUT_OF_MEMORY) note_refused(g, key);
    return st;
}

RefusedKey sliced_key(const maxk_graph* g, int dim, int val_bytes) { return {kRefusedSliced, sliced_copy_bytes(g->N, dim, val_bytes)}; }

// Partial rows of the items that default_chunk made shorter than 2048 entries, at the widest row (at most 32 MiB; see
// there), allocated by maxk_graph_create: most of these rows are whole at 2048 entries, and a call on such a graph needs
// no buffer then, so it may come for the first time while its stream is being captured.  Without the memory, later calls
// allocate what they need.
void short_item_workspace(maxk_graph* g)
{
    const int64_t slots = std::max(g->csr_items.n_slots, g->csc_items.n_slots);
    if (g->chunk >= 2048 || slots == 0 || slots > 8192) return;
    float* fresh = nullptr;
    if (hipMalloc((void**)&fresh, sizeof(float) * (size_t)(slots * MAXK_MAX_DIM)) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    g->d_partials = fresh;
    g->partial_floats = slots * MAXK_MAX_DIM;
}

maxk_status ensure_workspace(maxk_graph* g, int dim, int k)
{
    const int64_t need = std::max<int64_t>(g->csr_items.n_slots * (int64_t)dim, g->csc_items.n_slots * (int64_t)k);
    if (need <= g->partial_floats) return MAXK_OK;
    float* fresh = nullptr;
    MAXK_HIP_TRY(hipMalloc((void**)&fresh, sizeof(float) * (size_t)need));
    if (g->d_partials) {
        MAXK_HIP_TRY(hipDeviceSynchronize());  // nothing may still be using the old buffer
        (void)hipFree(g->d_partials);
    }
    g->d_partials = fresh;
    g->partial_floats = need;
    return MAXK_OK;
}

void free_slabs(SlabSet& S)
{
    (void)hipFree(S.d_src);
    (void)hipFree(S.d_val);
    (void)hipFree(S.d_visit_node);
    (void)hipFree(S.d_visit_begin);
    (void)hipFree(S.d_long_visit);
    std::free(S.h_slab_visit);
    std::free(S.h_slab_long);
    std::free(S.h_slab_lone);
    S = SlabSet();
}

// key[q] = slab(source of CSC position q) * N + destination of q;  iota[q] = q
__global__ __launch_bounds__(256) void slab_keys_kernel(const int32_t* __restrict__ csc_ptr,
                                                        const int32_t* __restrict__ csc_src, int64_t N, int64_t nnz,
                                                        int32_t slab_rows, uint64_t* __restrict__ key,
                                                        uint32_t* __restrict__ iota)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nnz; q += stride) {
        int64_t lo = 0, hi = N;  // largest j with csc_ptr[j] <= q
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)csc_ptr[mid] <= q) lo = mid; else hi = mid;
        }
        key[q] = (uint64_t)(csc_src[q] / slab_rows) * (uint64_t)N + (uint64_t)lo;
        iota[q] = (uint32_t)q;
    }
}

__global__ __launch_bounds__(256) void slab_gather_kernel(const uint32_t* __restrict__ perm,
                                                          const uint64_t* __restrict__ key_sorted,
                                                          const int32_t* __restrict__ csc_src,
                                                          const float* __restrict__ csc_val, int64_t nnz,
                                                          int32_t* __restrict__ out_src, float* __restrict__ out_val,
                                                          uint32_t* __restrict__ head)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nnz; r += stride) {
        const uint32_t q = perm[r];
        out_src[r] = csc_src[q];
        out_val[r] = csc_val[q];
        head[r] = (r == 0 || key_sorted[r] != key_sorted[r - 1]) ? 1u : 0u;
    }
}

// at every head position r (visit number v = rank[r] - 1): record the visit
__global__ __launch_bounds__(256) void slab_visits_kernel(const uint32_t* __restrict__ head,
                                                          const uint32_t* __restrict__ rank,
                                                          const uint64_t* __restrict__ key_sorted, int64_t N,
                                                          int64_t nnz, int32_t* __restrict__ visit_node,
                                                          int32_t* __restrict__ visit_begin,
                                                          int32_t* __restrict__ visit_slab)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nnz; r += stride) {
        if (!head[r]) continue;
        const uint32_t v = rank[r] - 1u;
        const uint64_t key = key_sorted[r];
        visit_node[v] = (int32_t)(key % (uint64_t)N);
        visit_slab[v] = (int32_t)(key / (uint64_t)N);
        visit_begin[v] = (int32_t)r;
    }
}

// slab_first[s] = first visit whose slab is >= s (slab_first pre-filled with n_visits)
__global__ __launch_bounds__(256) void slab_first_kernel(const int32_t* __restrict__ visit_slab, int64_t n_visits,
                                                         int64_t* __restrict__ slab_first)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n_visits; v += stride) {
        const int32_t sl = visit_slab[v];
        const int32_t prev = v ? visit_slab[v - 1] : -1;
        for (int32_t s = prev + 1; s <= sl; ++s) slab_first[s] = v;
    }
}

__global__ __launch_bounds__(256) void fill_i64_kernel(int64_t* __restrict__ p, int64_t n, int64_t value)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

// From how many entries on the row-accumulating slab kernel gives a visit a wavefront of its own: kSlabLongVisit or a power of
// two above it.  Lone visits fill the chip from the start of a launch on, which shortens it where its end was long visits that
// began late; but the longest visit then shares its CU with other long ones, and where it takes most of a launch by itself they
// delay it.  So the line follows its share: r = its entries over a resident wavefront's share (7168 of them) of the slab's; 0.04 r
// of its length, at most 0.3.  us, dim 256, k = 64, r: visits from 33 / 64 / 256 / 512 / 1024 / no visit alone: 115 M entries on 233 k nodes,
// fp32, 1.2 5384 / 5492 / 5806 / 5831 / 5827 / 5855; 60 M on 180 k, bf16, 5.3 3742 / 3738 / 3666 / 3633 / 3671 / 4375; 24 M on 60 k,
// bf16, 5.7 1516 / 1464 / 1427 / 1400 / 1391 / 1437; 28 M on 90 k, bf16, 11 3194 / 3142 / 3073 / 3051 / 2960 / 3134; 14 M on 60 k, fp32, 14.5
// 1893 / 1842 / 1789 / 1769 / 1772 / 1921.  Over 18 graphs in fp32 and bf16 the line is within 3 % of the best of these, 33 up to 9 % off.
int32_t lone_visit_line(int32_t longest, int64_t entries)
{
    const double share = 7168.0 * longest / (double)std::max<int64_t>(entries, 1), line = std::min(0.3, 0.04 * share) * longest;
    int32_t n = kSlabLongVisit;
    while (2.0 * n <= line) n *= 2;
    return n;
}

// Regroups A^T by slabs of `slab_rows` source rows (see SlabSet) into the empty set S.  Synchronises the device.
maxk_status build_slabs(maxk_graph* g, SlabSet& S, int32_t slab_rows)
{
    MAXK_HIP_TRY(hipDeviceSynchronize());
    const int64_t N = g->N, nnz = g->nnz;
    const int32_t n_slabs = (int32_t)((N + slab_rows - 1) / slab_rows);
    S.h_slab_visit = (int64_t*)std::calloc((size_t)n_slabs + 1, sizeof(int64_t));
    if (!S.h_slab_visit) return MAXK_OUT_OF_MEMORY;
    S.n_slabs = n_slabs;
    if (nnz == 0) {
        S.slab_rows = slab_rows;
        return MAXK_OK;
    }
    hipStream_t s = nullptr;
    uint64_t *d_key = nullptr, *d_key_sorted = nullptr;
    uint32_t *d_iota = nullptr, *d_perm = nullptr, *d_head = nullptr, *d_rank = nullptr;
    int32_t* d_visit_slab = nullptr;
    int64_t* d_slab_first = nullptr;
    void* d_tmp = nullptr;
    auto cleanup = [&]() {
        (void)hipFree(d_key); (void)hipFree(d_key_sorted); (void)hipFree(d_iota); (void)hipFree(d_perm);
        (void)hipFree(d_head); (void)hipFree(d_rank); (void)hipFree(d_visit_slab); (void)hipFree(d_slab_first);
        (void)hipFree(d_tmp);
    };
#define MAXK_TRY_CLEAN(expr)                                                           \
    do {                                                                               \
        hipError_t _e = (expr);                                                        \
        if (_e != hipSuccess) { cleanup(); free_slabs(S); return hip_fail(_e); }       \
    } while (0)
    // 8 spare entries at the end: the row-accumulating kernel fetches entries eight at a time with scalar loads
    MAXK_TRY_CLEAN(hipMalloc((void**)&S.d_src, sizeof(int32_t) * (size_t)(nnz + 8)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&S.d_val, sizeof(float) * (size_t)(nnz + 8)));
    MAXK_TRY_CLEAN(hipMemsetAsync(S.d_src + nnz, 0, sizeof(int32_t) * 8, s));
    MAXK_TRY_CLEAN(hipMemsetAsync(S.d_val + nnz, 0, sizeof(float) * 8, s));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_key, sizeof(uint64_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_key_sorted, sizeof(uint64_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_iota, sizeof(uint32_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_perm, sizeof(uint32_t) * (size_t)nnz));
    const unsigned blocks = (unsigned)std::min<int64_t>((nnz + 255) / 256, 65536);
    hipLaunchKernelGGL(slab_keys_kernel, dim3(blocks), dim3(256), 0, s, g->d_csc_ptr, g->d_csc_src, N, nnz, slab_rows,
                       d_key, d_iota);
    MAXK_TRY_CLEAN(hipGetLastError());
    int end_bit = 1;
    while (end_bit < 64 && ((uint64_t)1 << end_bit) < (uint64_t)n_slabs * (uint64_t)N) ++end_bit;
    size_t tmp_bytes = 0;
    MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(nullptr, tmp_bytes, d_key, d_key_sorted, d_iota, d_perm, (size_t)nnz, 0,
                                             (unsigned)end_bit, s));
    MAXK_TRY_CLEAN(hipMalloc(&d_tmp, tmp_bytes ? tmp_bytes : 16));
    MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(d_tmp, tmp_bytes, d_key, d_key_sorted, d_iota, d_perm, (size_t)nnz, 0,
                                             (unsigned)end_bit, s));
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
    (void)hipFree(d_tmp); d_tmp = nullptr;
    (void)hipFree(d_key); d_key = nullptr;
    (void)hipFree(d_iota); d_iota = nullptr;
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_head, sizeof(uint32_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_rank, sizeof(uint32_t) * (size_t)nnz));
    hipLaunchKernelGGL(slab_gather_kernel, dim3(blocks), dim3(256), 0, s, d_perm, d_key_sorted, g->d_csc_src,
                       g->d_csc_val, nnz, S.d_src, S.d_val, d_head);
    MAXK_TRY_CLEAN(hipGetLastError());
    tmp_bytes = 0;
    MAXK_TRY_CLEAN(rocprim::inclusive_scan(nullptr, tmp_bytes, d_head, d_rank, (size_t)nnz, rocprim::plus<uint32_t>(), s));
    MAXK_TRY_CLEAN(hipMalloc(&d_tmp, tmp_bytes ? tmp_bytes : 16));
    MAXK_TRY_CLEAN(rocprim::inclusive_scan(d_tmp, tmp_bytes, d_head, d_rank, (size_t)nnz, rocprim::plus<uint32_t>(), s));
    uint32_t n_visits32 = 0;
    MAXK_TRY_CLEAN(hipMemcpyAsync(&n_visits32, d_rank + (nnz - 1), sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
    const int64_t n_visits = n_visits32;
    MAXK_TRY_CLEAN(hipMalloc((void**)&S.d_visit_node, sizeof(int32_t) * (size_t)n_visits));
    MAXK_TRY_CLEAN(hipMalloc((void**)&S.d_visit_begin, sizeof(int32_t) * (size_t)(n_visits + 1)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_visit_slab, sizeof(int32_t) * (size_t)n_visits));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_slab_first, sizeof(int64_t) * (size_t)(n_slabs + 1)));
    hipLaunchKernelGGL(slab_visits_kernel, dim3(blocks), dim3(256), 0, s, d_head, d_rank, d_key_sorted, N, nnz,
                       S.d_visit_node, S.d_visit_begin, d_visit_slab);
    const int32_t nnz32 = (int32_t)nnz;
    MAXK_TRY_CLEAN(hipMemcpyAsync(S.d_visit_begin + n_visits, &nnz32, sizeof(int32_t), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(fill_i64_kernel, dim3((unsigned)((n_slabs + 1 + 255) / 256)), dim3(256), 0, s, d_slab_first,
                       (int64_t)n_slabs + 1, n_visits);
    hipLaunchKernelGGL(slab_first_kernel, dim3((unsigned)std::min<int64_t>((n_visits + 255) / 256, 65536)), dim3(256), 0,
                       s, d_visit_slab, n_visits, d_slab_first);
    MAXK_TRY_CLEAN(hipGetLastError());
    MAXK_TRY_CLEAN(hipMemcpyAsync(S.h_slab_visit, d_slab_first, sizeof(int64_t) * (size_t)(n_slabs + 1),
                                  hipMemcpyDeviceToHost, s));
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
    // long visits (hub destinations inside one slab): listed per slab on the host
    try {
        std::vector<int32_t> h_begin((size_t)n_visits + 1), h_long, in_order;
        MAXK_TRY_CLEAN(hipMemcpy(h_begin.data(), S.d_visit_begin, sizeof(int32_t) * (size_t)(n_visits + 1),
                                 hipMemcpyDeviceToHost));
        S.h_slab_long = (int64_t*)std::calloc((size_t)n_slabs + 1, sizeof(int64_t));
        S.h_slab_lone = (LoneVisits*)std::calloc((size_t)n_slabs, sizeof(LoneVisits));
        if (!S.h_slab_long || !S.h_slab_lone) { cleanup(); free_slabs(S); return MAXK_OUT_OF_MEMORY; }
        for (int32_t sl = 0; sl < n_slabs; ++sl) {
            S.h_slab_long[sl] = (int64_t)h_long.size();
            for (int64_t v = S.h_slab_visit[sl]; v < S.h_slab_visit[sl + 1]; ++v)
                if (h_begin[(size_t)v + 1] - h_begin[(size_t)v] > kSlabLongVisit) h_long.push_back((int32_t)v);
            // longest first, by powers of two (a list that is walked from its front by as many wavefronts as there are).  us of
            // the sampled kernel, in destination order / so: 79 M entries on 133 k nodes, k = 16 3578 / 3468; 7 M on 63 k,
            // width 99, k = 32 562 / 540; 14 M on 60 k, k = 16 1806 / 1756, but bf16, k = 8 1067 / 1093; 115 M on 233 k within 1 %.
            // Of the row-accumulating one: 18 M on 60 k, k = 32, bf16 839 / 720; 40 M on 100 k, dim 300, k = 100, bf16 3650 / 3518;
            // 14 M on 60 k, k = 64, bf16 1864 / 1941 (every long visit alone; the line of lone visits mends that).
            const auto first = h_long.begin() + S.h_slab_long[sl], last = h_long.end();
            const auto size_class = [&](int32_t v) { return std::countl_zero((uint32_t)(h_begin[(size_t)v + 1] - h_begin[(size_t)v])); };
            size_t at[33] = {};
            for (auto v = first; v != last; ++v) ++at[size_class(*v) + 1];
            for (int c = 0; c < 32; ++c) at[c + 1] += at[c];
            int32_t longest = 0;
            for (auto v = first; v != last; ++v) longest = std::max(longest, h_begin[(size_t)*v + 1] - h_begin[(size_t)*v]);
            const int32_t line = lone_visit_line(longest, h_begin[(size_t)S.h_slab_visit[sl + 1]] - h_begin[(size_t)S.h_slab_visit[sl]]);
            S.h_slab_lone[sl] = line <= kSlabLongVisit ? LoneVisits{kSlabLongVisit, (int32_t)(last - first)}
                                                       : LoneVisits{line - 1, (int32_t)at[std::countl_zero((uint32_t)line) + 1]};
            in_order.resize((size_t)(last - first));
            for (auto v = first; v != last; ++v) in_order[at[size_class(*v)]++] = *v;
            std::copy(in_order.begin(), in_order.end(), first);
        }
        S.h_slab_long[n_slabs] = (int64_t)h_long.size();
        S.n_long = (int64_t)h_long.size();
        if (S.n_long) {
            MAXK_TRY_CLEAN(hipMalloc((void**)&S.d_long_visit, sizeof(int32_t) * h_long.size()));
            MAXK_TRY_CLEAN(hipMemcpy(S.d_long_visit, h_long.data(), sizeof(int32_t) * h_long.size(), hipMemcpyHostToDevice));
        }
    } catch (const std::bad_alloc&) {
        cleanup();
        free_slabs(S);
        return MAXK_OUT_OF_MEMORY;
    }
#undef MAXK_TRY_CLEAN
    cleanup();
    S.n_visits = n_visits;
    S.slab_rows = slab_rows;
    return MAXK_OK;
}

// Slab height for hidden width `dim`: a slab of dY should sit comfortably inside one XCD's 4 MB L2.
int32_t slab_rows_for(const maxk_graph* g, int dim, int val_bytes = 4)
{
    const int64_t rows = (int64_t)g->slab_kb * 1024 / ((int64_t)dim * val_bytes);
    return (int32_t)std::max<int64_t>(rows, 64);
}

bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();  // the default stream while another one is being captured: nothing may be allocated either
    return true;
}

// The regrouping of A^T for one slab height: built on first use (or by maxk_graph_reserve*), then kept until the
// handle is destroyed, so alternating hidden widths or dY formats on one handle never rebuilds anything.
// existing_only(): asked where the table is missing; nothing is built then, and that is not remembered as a refusal.
template <class F>
maxk_status slabs_for(maxk_graph* g, int32_t slab_rows, const F& existing_only, SlabSet** out)
{
    for (SlabSet* S : g->slab_cache)
        if (S->slab_rows == slab_rows) { *out = S; return MAXK_OK; }
    if (existing_only()) return MAXK_OUT_OF_MEMORY;
    SlabSet* S = new (std::nothrow) SlabSet();
    maxk_status st = MAXK_OUT_OF_MEMORY;
    if (S && !denied(g, g->nnz * 8)) {
        try {
            st = build_slabs(g, *S, slab_rows);
            if (st == MAXK_OK) g->slab_cache.push_back(S);
        } catch (const std::bad_alloc&) {
            st = MAXK_OUT_OF_MEMORY;
        }
    }
    if (st != MAXK_OK) {
        if (S) free_slabs(*S);
        delete S;
        if (st == MAXK_OUT_OF_MEMORY) note_refused(g, {kRefusedSlab, slab_rows});
        return st;
    }
    *out = S;
    return MAXK_OK;
}

RefusedKey tiled_key(const TiledShape& sh, int k) { return {kRefusedTiled, sh.D, sh.TR, k / tiled_positions_per_lane(k)}; }

template <class F>
maxk_status tiled_for(maxk_graph* g, int dim, int k, const F& existing_only, TiledSet** out)
{
    TiledShape sh;
    if (!tiled_shape(g->N, g->nnz, dim, k, sh)) return MAXK_UNSUPPORTED;
    for (TiledSet* T : g->tiled_cache)
        if (T->D == sh.D && T->TR == sh.TR && T->LPV == k / tiled_positions_per_lane(k)) { *out = T; return MAXK_OK; }
    if (existing_only()) return MAXK_OUT_OF_MEMORY;
    TiledSet* T = new (std::nothrow) TiledSet();
    maxk_status st = MAXK_OUT_OF_MEMORY;
    if (T && !denied(g, g->nnz * 8)) {
        try {
            st = build_tiled(*T, g->N, g->nnz, g->d_csc_ptr, g->d_csc_src, g->d_csc_val, sh.D, sh.TR, k);
            if (st == MAXK_OK) g->tiled_cache.push_back(T);
        } catch (const std::bad_alloc&) {
            st = MAXK_OUT_OF_MEMORY;
        }
    }
    if (st != MAXK_OK) {
        if (T) free_tiled(*T);
        delete T;
        if (st == MAXK_OUT_OF_MEMORY) note_refused(g, tiled_key(sh, k));
        return st;
    }
    *out = T;
    return MAXK_OK;
}

bool regs_refused(const maxk_graph* g, const RegsShape& sh)
{
    return std::find(g->regs_refused.begin(), g->regs_refused.end(), sh) != g->regs_refused.end();
}

template <class F>
maxk_status regs_for(maxk_graph* g, const RegsShape& sh, const F& existing_only, RegsSet** out)
{
    for (RegsSet* T : g->regs_cache)
        if (T->shape == sh) { *out = T; return MAXK_OK; }
    if (existing_only()) return MAXK_OUT_OF_MEMORY;
    RegsSet* T = new (std::nothrow) RegsSet();
    maxk_status st = MAXK_OUT_OF_MEMORY;
    if (T && !denied(g, g->nnz * 8)) {
        try {
            st = build_regs(*T, sh, g->N, g->nnz, g->d_rowptr, g->d_csc_ptr, g->d_csc_src, g->d_csc_val);
            if (st == MAXK_OK) g->regs_cache.push_back(T);
        } catch (const std::bad_alloc&) {
            st = MAXK_OUT_OF_MEMORY;
        }
    }
    if (st != MAXK_OK) {
        if (T) free_regs(*T);
        delete T;
        if (st != MAXK_HIP_ERROR && !regs_refused(g, sh)) {  // lack of memory, or a graph that the lists do not hold
            try {
                g->regs_refused.push_back(sh);
            } catch (const std::bad_alloc&) {  // then the next call tries again
            }
        }
        return st;
    }
    *out = T;
    return MAXK_OK;
}

void free_sweep(SweepSet& W)
{
    (void)hipFree(W.d_ent);
    (void)hipFree(W.d_batch);
    (void)hipFree(W.d_rows);
    W = SweepSet();
}

// `count` consecutive work items that become row `row` of consecutive bins
struct SweepRun { uint32_t item, bin, count, row; };

// Deals the work items to bins of per_bin rows, longest first, each to the bin with the fewest entries so far that has a row
// left (in rounds of one item a bin the fullest bins stay up to 20 % above the mean, and the forward pass takes 5 % longer
// at four rows a bin).  Bins of equal load are moved a run at a time, so the work follows the number of different lengths
// and not of items.  The runs come in the order of their items.
void sweep_deal(const std::vector<std::pair<int32_t, int64_t>>& lengths, int64_t n_bins, int per_bin, std::vector<SweepRun>& runs)
{
    std::map<int64_t, std::deque<SweepRun>> open;  // by load: bins in runs, `row` = rows taken so far
    open[0].push_back({0, 0, (uint32_t)n_bins, 0});
    uint32_t item = 0;
    for (const auto& [len, times] : lengths) {
        for (int64_t left = times; left > 0;) {
            const auto least = open.begin();
            const int64_t load = least->first;
            SweepRun& bins = least->second.front();
            const SweepRun run = {item, bins.bin, (uint32_t)std::min<int64_t>(left, bins.count), bins.row};
            bins.bin += run.count;
            bins.count -= run.count;
            if (bins.count == 0) {
                least->second.pop_front();
                if (least->second.empty()) open.erase(least);
            }
            if ((int)run.row + 1 < per_bin) open[load + len].push_back({0, run.bin, run.count, run.row + 1});
            runs.push_back(run);
            item += run.count;
            left -= run.count;
        }
    }
}

// item_at[place] = the work item of every row of every bin (place = bin * per_bin + row; -1 from the caller: none), and back
__global__ __launch_bounds__(256) void sweep_places_kernel(const SweepRun* __restrict__ runs, int n_runs, int64_t n_items,
                                                           int per_bin, uint32_t* __restrict__ place, uint32_t* __restrict__ item_at)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_items; i += stride) {
        int lo = 0, hi = n_runs;  // the last run that starts at or before item i
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if ((int64_t)runs[mid].item <= i) lo = mid; else hi = mid;
        }
        const SweepRun r = runs[lo];
        const uint32_t at = (r.bin + ((uint32_t)i - r.item)) * (uint32_t)per_bin + r.row;
        place[i] = at;
        item_at[at] = (uint32_t)i;
    }
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t* __restrict__ p, int64_t n, uint32_t x)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = x;
}

// The entries that a sweep gives a work item: first, first + stride, ...  A piece of a split row takes every n-th entry of the
// row and not a run of them: a run covers a part of the source nodes only, and its bin would be ahead of or behind the others
// on their way over them all along.  us, runs / every n-th: 115 M entries on 233 k nodes k = 32 2059 / 2020, k = 64
// 3149 / 2979, k = 128 6811 / 6022; 43 M on 576 k k = 64 2060 / 1918; 126 M on 2.4 M k = 64 4838 / 4561.
struct SweepItem { int32_t first, stride, count; };
__device__ SweepItem sweep_item(const WorkItem it, const SplitRow* __restrict__ split, int n_split, const int32_t* __restrict__ ptr)
{
    if (it.slot < 0) return {it.begin, 1, it.end - it.begin};
    int lo = 0, hi = n_split;  // the last split row that starts at or before the slot
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (split[mid].slot_begin <= it.slot) lo = mid; else hi = mid;
    }
    const int32_t pieces = split[lo].slot_count, piece = it.slot - split[lo].slot_begin, begin = ptr[it.row];
    return {begin + piece, pieces, (ptr[it.row + 1] - begin - piece + pieces - 1) / pieces};
}

// Rows and partial-sum slots of every bin, entries of every (bin, lane group), batches of every bin.  Each row's own entries
// take the lane groups in turn: dealt by their place in the bin, the entries of two rows with the same neighbours alternate
// and each row would end up in one lane group, one running sum.
__global__ __launch_bounds__(256) void sweep_bins_kernel(const WorkItem* __restrict__ items, const SplitRow* __restrict__ split,
                                                         int n_split, const int32_t* __restrict__ ptr,
                                                         const uint32_t* __restrict__ item_at,
                                                         int64_t n_bins, int per_bin, uint32_t groups, uint32_t batch_len,
                                                         int2* __restrict__ rows, uint32_t* __restrict__ list_len,
                                                         uint32_t* __restrict__ batches)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n_bins; b += stride) {
        for (uint32_t g = 0; g < groups; ++g) list_len[b * groups + g] = 0;
        for (int r = 0; r < per_bin; ++r) {
            const uint32_t i = item_at[b * per_bin + r];
            const WorkItem it = i != 0xFFFFFFFFu ? items[i] : WorkItem{-1, 0, 0, -1};
            rows[b * per_bin + r] = make_int2(it.row, it.slot);
            const uint32_t len = (uint32_t)sweep_item(it, split, n_split, ptr).count;
            for (uint32_t j = 0; j < groups; ++j)  // entries j, j + groups, ... of the row
                list_len[b * groups + (j + (uint32_t)r) % groups] += (len + groups - 1 - j) / groups;
        }
        uint32_t longest = 0;
        for (uint32_t g = 0; g < groups; ++g) longest = max(longest, list_len[b * groups + g]);
        batches[b] = (longest + batch_len - 1) / batch_len;
    }
}

// key[p] = (bin, lane group) << 32 | source node, payload[p] = p, row_of[p] = row of the bin, for the entries of every work
// item.  Workgroups stride over the items: one each would be 2^32 threads, more than a launch holds, from 2^24 items up.
__global__ __launch_bounds__(256) void sweep_keys_kernel(const WorkItem* __restrict__ items, const SplitRow* __restrict__ split,
                                                         int n_split, const int32_t* __restrict__ ptr,
                                                         const uint32_t* __restrict__ place,
                                                         int64_t n_items, uint32_t per_bin, uint32_t groups,
                                                         const int32_t* __restrict__ col, uint64_t* __restrict__ key,
                                                         uint32_t* __restrict__ entry, uint8_t* __restrict__ row_of)
{
    for (int64_t i = blockIdx.x; i < n_items; i += gridDim.x) {
        const SweepItem it = sweep_item(items[i], split, n_split, ptr);
        const uint32_t row = place[i] % per_bin;
        const uint64_t bin = place[i] / per_bin;
        for (int e = (int)threadIdx.x; e < it.count; e += blockDim.x) {
            const int64_t p = it.first + (int64_t)e * it.stride;
            key[p] = (bin * groups + ((uint32_t)e + row) % groups) << 32 | (uint32_t)col[p];
            entry[p] = (uint32_t)p;
            row_of[p] = (uint8_t)row;
        }
    }
}

__global__ __launch_bounds__(256) void sweep_fill_kernel(int2* __restrict__ ent, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) ent[i] = make_int2(-1, 0);
}

__global__ __launch_bounds__(256) void sweep_entries_kernel(const uint64_t* __restrict__ key, const uint32_t* __restrict__ entry,
                                                            const uint8_t* __restrict__ row_of, const float* __restrict__ val,
                                                            int64_t nnz, const uint32_t* __restrict__ list_first,
                                                            const uint32_t* __restrict__ batch, uint32_t groups,
                                                            uint32_t batch_len, int2* __restrict__ ent)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nnz; i += stride) {
        const uint32_t list = (uint32_t)(key[i] >> 32), bin = list / groups, g = list % groups, p = entry[i];
        const uint32_t n = (uint32_t)i - list_first[list];
        ent[(((int64_t)batch[bin] + n / batch_len) * groups + g) * batch_len + n % batch_len] =
            make_int2((int)((uint32_t)key[i] | (uint32_t)row_of[p] << kSweepRowShift), __float_as_int(val[p]));
    }
}

// Deals the work items to bins and lays their entries out.  Synchronises the device.
maxk_status build_sweep(maxk_graph* g, SweepSet& W, int groups, int batch_len, int per_bin)
{
    MAXK_HIP_TRY(hipDeviceSynchronize());
    const int64_t n_items = g->csr_items.n_items, nnz = g->nnz, n_bins = (n_items + per_bin - 1) / per_bin, n_lists = n_bins * groups;
    std::vector<SweepRun> runs;
    sweep_deal(g->csr_lengths, n_bins, per_bin, runs);
    hipStream_t s = nullptr;
    uint64_t *d_key = nullptr, *d_key_sorted = nullptr;
    uint32_t *d_entry = nullptr, *d_perm = nullptr, *d_list_len = nullptr, *d_list_first = nullptr, *d_batches = nullptr,
             *d_place = nullptr, *d_item_at = nullptr;
    SweepRun* d_runs = nullptr;
    uint8_t* d_row_of = nullptr;
    void* d_tmp = nullptr;
    auto cleanup = [&]() {
        (void)hipFree(d_key); (void)hipFree(d_key_sorted); (void)hipFree(d_entry); (void)hipFree(d_perm);
        (void)hipFree(d_list_len); (void)hipFree(d_list_first); (void)hipFree(d_batches); (void)hipFree(d_row_of); (void)hipFree(d_tmp);
        (void)hipFree(d_place); (void)hipFree(d_item_at); (void)hipFree(d_runs);
    };
#define MAXK_TRY_CLEAN(expr)                                                           \
    do {                                                                               \
        hipError_t _e = (expr);                                                        \
        if (_e != hipSuccess) { cleanup(); free_sweep(W); return hip_fail(_e); }       \
    } while (0)
    // (fewer than 2^31 / 8 + 2 * 2^26 batches: a bin has at most one more than its entries fill)
    MAXK_TRY_CLEAN(hipMalloc((void**)&W.d_batch, sizeof(uint32_t) * (size_t)(n_bins + 1)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&W.d_rows, sizeof(int2) * (size_t)(n_bins * per_bin)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_batches, sizeof(uint32_t) * (size_t)(n_bins + 1)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_list_len, sizeof(uint32_t) * (size_t)n_lists));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_list_first, sizeof(uint32_t) * (size_t)n_lists));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_place, sizeof(uint32_t) * (size_t)n_items));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_item_at, sizeof(uint32_t) * (size_t)(n_bins * per_bin)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_runs, sizeof(SweepRun) * runs.size()));
    MAXK_TRY_CLEAN(hipMemcpy(d_runs, runs.data(), sizeof(SweepRun) * runs.size(), hipMemcpyHostToDevice));
    size_t tmp_bytes = 0, scan_bytes = 0;
    MAXK_TRY_CLEAN(rocprim::exclusive_scan(nullptr, tmp_bytes, d_batches, W.d_batch, 0u, (size_t)(n_bins + 1), rocprim::plus<uint32_t>(), s));
    MAXK_TRY_CLEAN(rocprim::exclusive_scan(nullptr, scan_bytes, d_list_len, d_list_first, 0u, (size_t)n_lists, rocprim::plus<uint32_t>(), s));
    tmp_bytes = std::max<size_t>({tmp_bytes, scan_bytes, 16});
    MAXK_TRY_CLEAN(hipMalloc(&d_tmp, tmp_bytes));
    const dim3 bin_blocks((unsigned)std::min<int64_t>((n_bins + 255) / 256, 65536));
    hipLaunchKernelGGL(fill_u32_kernel, bin_blocks, dim3(256), 0, s, d_item_at, n_bins * per_bin, 0xFFFFFFFFu);
    hipLaunchKernelGGL(sweep_places_kernel, bin_blocks, dim3(256), 0, s, d_runs, (int)runs.size(), n_items, per_bin, d_place, d_item_at);
    MAXK_TRY_CLEAN(hipGetLastError());
    hipLaunchKernelGGL(sweep_bins_kernel, bin_blocks, dim3(256), 0, s, g->csr_items.d_items, g->csr_items.d_split,
                       (int)g->csr_items.n_split, g->d_rowptr, d_item_at, n_bins, per_bin, (uint32_t)groups, (uint32_t)batch_len, W.d_rows, d_list_len, d_batches);
    MAXK_TRY_CLEAN(hipGetLastError());
    scan_bytes = tmp_bytes;
    MAXK_TRY_CLEAN(rocprim::exclusive_scan(d_tmp, scan_bytes, d_batches, W.d_batch, 0u, (size_t)(n_bins + 1), rocprim::plus<uint32_t>(), s));
    scan_bytes = tmp_bytes;
    MAXK_TRY_CLEAN(rocprim::exclusive_scan(d_tmp, scan_bytes, d_list_len, d_list_first, 0u, (size_t)n_lists, rocprim::plus<uint32_t>(), s));
    uint32_t n_batches = 0;
    MAXK_TRY_CLEAN(hipMemcpyAsync(&n_batches, W.d_batch + n_bins, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
    (void)hipFree(d_tmp); d_tmp = nullptr;
    const int64_t n_ent = (int64_t)n_batches * groups * batch_len;
    MAXK_TRY_CLEAN(hipMalloc((void**)&W.d_ent, sizeof(int2) * (size_t)std::max<int64_t>(n_ent, 1)));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_key, sizeof(uint64_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_key_sorted, sizeof(uint64_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_entry, sizeof(uint32_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_perm, sizeof(uint32_t) * (size_t)nnz));
    MAXK_TRY_CLEAN(hipMalloc((void**)&d_row_of, (size_t)nnz));
    const unsigned blocks = (unsigned)std::min<int64_t>((nnz + 255) / 256, 65536);
    hipLaunchKernelGGL(sweep_keys_kernel, dim3((unsigned)std::min<int64_t>(n_items, 1 << 20)), dim3(256), 0, s,
                       g->csr_items.d_items, g->csr_items.d_split, (int)g->csr_items.n_split, g->d_rowptr, d_place, n_items,
                       (uint32_t)per_bin, (uint32_t)groups, g->d_col, d_key, d_entry, d_row_of);
    MAXK_TRY_CLEAN(hipGetLastError());
    int end_bit = 33;
    while (end_bit < 64 && ((uint64_t)1 << (end_bit - 32)) < (uint64_t)n_lists) ++end_bit;
    tmp_bytes = 0;
    MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(nullptr, tmp_bytes, d_key, d_key_sorted, d_entry, d_perm, (size_t)nnz, 0, (unsigned)end_bit, s));
    MAXK_TRY_CLEAN(hipMalloc(&d_tmp, tmp_bytes ? tmp_bytes : 16));
    MAXK_TRY_CLEAN(rocprim::radix_sort_pairs(d_tmp, tmp_bytes, d_key, d_key_sorted, d_entry, d_perm, (size_t)nnz, 0, (unsigned)end_bit, s));
    hipLaunchKernelGGL(sweep_fill_kernel, dim3(blocks), dim3(256), 0, s, W.d_ent, n_ent);
    hipLaunchKernelGGL(sweep_entries_kernel, dim3(blocks), dim3(256), 0, s, d_key_sorted, d_perm, d_row_of, g->d_val, nnz, d_list_first,
                       W.d_batch, (uint32_t)groups, (uint32_t)batch_len, W.d_ent);
    MAXK_TRY_CLEAN(hipGetLastError());
    MAXK_TRY_CLEAN(hipStreamSynchronize(s));
#undef MAXK_TRY_CLEAN
    cleanup();
    W.groups = groups;
    W.batch_len = batch_len;
    W.per_bin = per_bin;
    W.n_bins = n_bins;
    return MAXK_OK;
}

// Forward calls within a reserved shape build nothing; the others build what they need on first use.
bool reserved_for(const maxk_graph* g, int dim, int k)
{
    return std::any_of(g->reserved.begin(), g->reserved.end(), [=](const auto& r) { return dim <= r.first && k <= r.second; });
}

maxk_status note_reserved(maxk_graph* g, int dim, int k)
{
    if (reserved_for(g, dim, k)) return MAXK_OK;
    try {
        std::erase_if(g->reserved, [=](const auto& r) { return r.first <= dim && r.second <= k; });
        g->reserved.emplace_back(dim, k);
    } catch (const std::bad_alloc&) {
        return MAXK_OUT_OF_MEMORY;
    }
    return MAXK_OK;
}

// existing_only: nothing is built, and a refusal is not remembered (the call is being captured, or was reserved); bins of other
// numbers of rows do then, as long as a workgroup has a few wavefronts.  They do as well once the handle holds as many regroupings as there are
// splits into lane groups, 8 bytes an entry each: one split at three widths would be three of them, all splits fourteen.  (Bins that are too long for a
// width, built for narrower rows, are joined by others, up to twice as many; then such calls run row by row.)
constexpr size_t kSweepTables = 4;
maxk_status sweep_for(maxk_graph* g, int k, int dim, int per_bin, bool existing_only, SweepSet** out)
{
    const int groups = sweep_groups(k), batch_len = sweep_batch(k);
    for (SweepSet* W : g->sweep_cache)
        if (W->groups == groups && W->batch_len == batch_len && W->per_bin == per_bin) { *out = W; return MAXK_OK; }
    if (existing_only || g->sweep_cache.size() >= kSweepTables)
        for (SweepSet* W : g->sweep_cache)
            if (W->groups == groups && W->batch_len == batch_len && sweep_waves(k, W->per_bin, dim) >= 4) { *out = W; return MAXK_OK; }
    const RefusedKey key = {kRefusedSweep, groups, batch_len, per_bin};
    if (existing_only || g->sweep_cache.size() >= 2 * kSweepTables || is_refused(g, key)) return MAXK_UNSUPPORTED;
    SweepSet* W = new (std::nothrow) SweepSet();
    maxk_status st = MAXK_OUT_OF_MEMORY;
    if (W && !denied(g, g->nnz * 8)) {
        try {
            st = build_sweep(g, *W, groups, batch_len, per_bin);
            if (st == MAXK_OK) g->sweep_cache.push_back(W);
        } catch (const std::bad_alloc&) {
            st = MAXK_OUT_OF_MEMORY;
        }
    }
    if (st != MAXK_OK) {
        if (W) free_sweep(*W);
        delete W;
        note_refused(g, key);
        return st;
    }
    *out = W;
    return MAXK_OK;
}

// The forward kernel repacks the CBSR when a row of it is well below a cache line - but for one that an L2 has room for beside the
// entries: there a launch more costs what the requests gain.  us, repacked / not: 1 k nodes, k = 8 7.4 / 3.9; 4 k, 2.1 M entries,
// k = 16 24.4 / 21.6; 40 k, 1.2 M, k = 13 (2.6 MB) 31.7 / 25.8; 60 k, 3.6 M, k = 8 (2.4 MB) 47.7 / 49.0; 60 k, 18 M, k = 16 (4.8
// MB) 128 / 172; 132 k, 79 M, k = 8 (5.3 MB) 700 / 979.
constexpr int64_t kFwdPackFrom = 3 << 20;  // bytes of the CBSR
bool fwd_uses_packed(const maxk_graph* g, int k, int index_bytes, int val_bytes)
{
    if (fwd_layout(k, index_bytes, val_bytes) == kFwdArrays) return false;  // no kernel reads such records
    const int row = k * (val_bytes + index_bytes);
    return g->fwd_pack_max >= 0 ? row <= g->fwd_pack_max : row <= 96 && g->N * (int64_t)row > kFwdPackFrom;
}

// Rows of a bin of the forward sweep for MaxK k, 0 where the row-by-row kernel is taken.  The sweep pays when the CBSR is
// several times an L2, the bins fill the chip (256 CUs x 16 wavefronts), and a bin has enough entries for its padding to whole
// batches and its copies of the rows.  The lines are drawn by lane groups and row size where both sides were measured, over 11 graphs of
// 30 k to 2 M nodes, average degree 15 to 500, k 8 to 128, widths 64 to 512 (profiles/forward_sweep_rule_over_graphs.txt: the kernel
// taken is 0.3 % above the better one on average, 15 % at most, row by row 12 %, the sweep 9 % on average); us, row by row / sweep (MB: of the CBSR; entries: of a lane group):
//   8 groups: k = 8, 9.6 MB, 61 entries 715 / 649, 6.4 MB, 38 entries 275 / 290
//   4 groups: k = 16, 13 MB, 150 entries 433 / 332, 32 MB, 60 entries 406 / 398, 128 MB, 26 entries 2389 / 2378 (bf16), 256 MB, 26 entries 2426 / 2527;
//     k = 50, 62 MB, 60 entries 1603 / 1532, 25 MB, 20 entries 181 / 200
//   2 groups: k = 32, 40 MB, 301 entries 734 / 593, 16 MB, 102 entries 84 / 87, 96 MB, 40 entries 308 / 296; dim 512, 115 MB, 20 entries 396 / 471;
//     bf16 values 77 MB, 152 entries 707 / 669, 32 MB, 301 entries 418 / 432; k = 96, 14 MB, 149 entries 85 / 83, 346 MB, 27 entries 762 / 805
//   1 group: k = 64, 19 MB, 755 entries 297 / 255, bf16 19 MB, 205 entries 104 / 115, 192 MB, 80 entries 456 / 403; k = 128, dim 512, 77 MB, 205 entries
//     360 / 289, 23 MB, 298 entries 108 / 127
int sweep_rows(const maxk_graph* g, int dim, int k, int index_bytes, int val_bytes)
{
    if (!sweep_takes(k) || dim > 512 || g->N > (1 << kSweepRowShift) || g->nnz == 0 || g->fwd_sweep == 1) return 0;
    const int per_bin = sweep_bin_rows(k, dim), groups = sweep_groups(k);
    // a wavefront per bin, rounded up to whole workgroups, is below the 2^32 threads of a launch
    if ((g->csr_items.n_items + per_bin - 1) / per_bin > (1 << 26) - 64) return 0;
    if (g->fwd_sweep == 2) return per_bin;
    const int record = fwd_uses_packed(g, k, index_bytes, val_bytes) ? fwd_packed_record_bytes(k, index_bytes, val_bytes)
                                                                     : k * (val_bytes + index_bytes);
    const double bins = (double)g->csr_items.n_items / per_bin, table = (double)g->N * record;
    const double entries = (double)g->nnz / (bins * groups) * std::min(1.0, 256.0 / dim);  // of a lane group, by the length of its rows
    const bool pays = groups == 8   ? table >= 8e6 && entries >= 48.0
                      : groups == 4 ? (table >= 9e6 && entries >= 100.0) || (table >= 20e6 && entries >= 58.0)
                      : groups == 1 ? table >= 18e6 && entries >= 60.0
                      : k > kWave   ? table >= 14e6 && entries >= 32.0
                      : val_bytes == 4 ? (table >= 10e6 && entries >= 300.0) || (table >= 20e6 && entries >= 40.0)
                                       : (table >= 10e6 && entries >= 500.0) || (table >= 60e6 && entries >= 60.0);
    return pays && bins >= 4096.0 ? per_bin : 0;
}

maxk_status ensure_packed(maxk_graph* g, int k, int index_bytes, int val_bytes)
{
    const int64_t need = g->N * (int64_t)fwd_packed_record_bytes(k, index_bytes, val_bytes);
    if (need <= g->packed_bytes) return MAXK_OK;
    char* fresh = nullptr;
    MAXK_HIP_TRY(hipMalloc((void**)&fresh, (size_t)need));
    if (g->d_packed) {
        MAXK_HIP_TRY(hipDeviceSynchronize());
        (void)hipFree(g->d_packed);
    }
    g->d_packed = fresh;
    g->packed_bytes = need;
    return MAXK_OK;
}

// A copy that has become too small is kept until the handle is destroyed: pull needs no other buffer on a graph without
// split rows, and a captured backward pass of a narrower dY may be replayed after this.
maxk_status ensure_sliced(maxk_graph* g, int dim, int val_bytes)
{
    const int64_t need = sliced_copy_bytes(g->N, dim, val_bytes);
    if (need <= g->sliced_bytes) return MAXK_OK;
    try {
        g->sliced_before.reserve(g->sliced_before.size() + 1);
    } catch (const std::bad_alloc&) {
        return MAXK_OUT_OF_MEMORY;
    }
    char* fresh = nullptr;
    const maxk_status st = allocate(g, (void**)&fresh, need, sliced_key(g, dim, val_bytes));
    if (st != MAXK_OK) return st;
    if (g->d_sliced) {
        g->sliced_before.push_back(g->d_sliced);
        g->sliced_before_bytes += g->sliced_bytes;
    }
    g->d_sliced = fresh;
    g->sliced_bytes = need;
    return MAXK_OK;
}

maxk_status ensure_expand(maxk_graph* g, int k)
{
    const int64_t need = g->nnz * (int64_t)k;
    if (need <= g->expand_floats) return MAXK_OK;
    float* fresh = nullptr;
    const maxk_status st = allocate(g, (void**)&fresh, need * (int64_t)sizeof(float), {kRefusedExpand, k});
    if (st != MAXK_OK) return st;
    if (g->d_expand) {
        MAXK_HIP_TRY(hipDeviceSynchronize());
        (void)hipFree(g->d_expand);
    }
    g->d_expand = fresh;
    g->expand_floats = need;
    return MAXK_OK;
}

// hot_share[i] = share of the entries in the 2^i longest rows (1 once every row is counted).  Linear in N: rows are
// counted per length, lengths above the table's end one by one.
void hot_source_shares(const std::vector<int32_t>& rowptr, int64_t n, int64_t nnz, float (&share)[33])
{
    constexpr int kTable = 1 << 16;
    std::vector<int64_t> count(kTable, 0);
    std::vector<int32_t> longer;
    for (int64_t i = 0; i < n; ++i) {
        const int32_t len = rowptr[(size_t)i + 1] - rowptr[(size_t)i];
        if (len < kTable) ++count[(size_t)len]; else longer.push_back(len);
    }
    std::sort(longer.begin(), longer.end(), [](int32_t a, int32_t b) { return a > b; });
    int64_t rows = 0, entries = 0;
    int step = 0;  // share[0..step) are known
    const auto take = [&](int64_t len, int64_t times) {
        while (times > 0 && step < 33) {
            const int64_t now = std::min(times, ((int64_t)1 << step) - rows);
            rows += now;
            entries += now * len;
            times -= now;
            if (rows == (int64_t)1 << step) share[step++] = (float)((double)entries / (double)std::max<int64_t>(nnz, 1));
        }
    };
    for (int32_t len : longer) take(len, 1);
    for (int len = kTable - 1; len > 0; --len)
        if (count[(size_t)len]) take(len, count[(size_t)len]);
    while (step < 33) share[step++] = 1.f;
}

// Share of the entries whose source is one of the `rows` most frequent ones: what a cache of that many rows can hit.
double hot_share(const maxk_graph* g, double rows)
{
    if (rows <= 1.0) return g->hot_share[0];
    const double at = std::min(31.999, std::log2(rows));
    const int i = (int)at;
    return g->hot_share[i] + (std::exp2(at - i) - 1.0) * (g->hot_share[i + 1] - g->hot_share[i]);
}

// Expected 128-byte lines of a dY row that k sorted columns touch
double lines_touched(int dim, int k, int val_bytes)
{
    const double per_line = 128.0 / val_bytes;
    return dim <= per_line ? 1.0 : (dim / per_line) * (1.0 - std::pow(1.0 - per_line / dim, (double)k));
}

// Whether the pull of whole rows works by units (bwd_pull_small_kernel, _wide_kernel), not by lane groups; `beyond`: share of the entries whose row is
// not among the most frequent 4 MB of them.  By lane groups an entry takes a third of the instructions; but the faster a wavefront walks its entries,
// the less the wavefronts keep together on their way over the sources, and rows that they shared in an L2 come from beyond it instead (8 k nodes, 0.8 M
// entries, rows of 2 KB, k = 32: 0.45 / 0.95 GB fetched, 8.8 / 4.1 M hits, 80 / 130 us).  So units are taken where an entry's lines, most of them from
// beyond L2, weigh more than its instructions.  us, units / lane groups, rows of 4-byte elements but *: k = 16, 8 k nodes, degree 101, 1 KB 37 / 49; 20 k, 61, 1 KB
// 73 / 82; 100 k, 61, 512 bytes* 289 / 319; 40 k, 31, 400 bytes (k = 13) 51 / 49; 300 k, 61, 256 bytes* (k = 12) 475 / 544; 300 k, 17, 256 bytes 167 / 132; k = 24, 8 k,
// 501, 2 KB 301 / 516; 60 k, 201, 768 bytes* 663 / 793; k = 64, 14 k, 29, 1 KB 35 / 46; 150 k, 121, 1 KB 1704 / 2157; 20 k, 61, 1 KB 125 / 90; k = 100, 12 k, 101,
// 2 KB 187 / 252; k = 128, 100 k, 61, 2 KB 1623 / 1437.  Over 966 such calls the kernel taken is 0.6 % above the better one on
// average, 16 % at most, lane groups everywhere 4.3 and 74 % (profiles/pull_by_units_and_by_lane_groups.txt).
// (16 < k <= 32 and a dY of several L2s together: 100 k nodes, degree 100 1043 / 1094, 169 k, 14 343 / 353, 1 M, 15 2361 / 2410.)
bool pull_by_units(int dim, int k, int val_bytes, int64_t N, int64_t nnz, double beyond)
{
    if (k < 9 || k > 128) return true;
    const double bytes = (double)N * dim * val_bytes, degree = (double)nnz / (double)std::max<int64_t>(N, 1);
    const double lines = lines_touched(dim, k, val_bytes) * (5.0 + 12.0 * beyond);  // ps an entry
    if (k <= 16) return beyond >= 0.25 && (lines > 40.0 || (degree >= 60.0 && beyond >= 0.33));
    if (k <= 32) return bytes > (64 << 20) || (beyond >= 0.25 && lines > 60.0) || (degree >= 100.0 && beyond >= 0.5);
    if (k <= 64) return beyond >= 0.52 && lines > 70.0 && (degree >= 40.0 || bytes < 64e6);
    return beyond >= 0.5 && lines > 140.0 && bytes < 35e6;
}

bool pull_by_units(const maxk_graph* g, int dim, int k, int val_bytes)
{
    return pull_by_units(dim, k, val_bytes, g->N, g->nnz, 1.0 - hot_share(g, 4e6 / ((double)dim * val_bytes)));
}

// The same of the destinations that the register-tiled kernel leaves, with fewest in-entries: nothing that wavefronts could keep together over
// (2.4 M nodes, k = 64, a whole pass: 12.24 ms by units, 11.96 by lane groups).
bool pull_tail_by_units(const maxk_graph* g, int dim, int k, int val_bytes) { return k <= 32 && pull_by_units(dim, k, val_bytes, g->N, g->nnz, 0.0); }

// The two forms of the pull over CSC, in seconds (see auto_bwd_mode for where the figures come from).  Whole rows are priced as the kernels by
// units take them; by lane groups (pull_by_units) they take down to 0.4 of that where the rows sit in L2, so that another kernel may be taken where
// they would be faster: 10 k nodes, degree 300, width 200, k = 24: sliced 139 us, whole rows by units 153, by lane groups 106.
// Plain: a line costs 5 ps when its row sits in L2 (4 MB of the most frequent rows), 17 ps when it does not; below that
// the gather's own instructions (12 + 0.55 k ps an entry).  One wavefront walks an item of at most `chunk` entries, 4 loads
// at a time and 0.6 us a round: the tail of small graphs.
// Column-sliced: every line of the row is gathered, 7 ps from L2 (24 thousand of the most frequent rows: a slice of 32
// thousand fills it) and 25 ps from beyond; 60 + 0.5 k ps per (item, slice) to sample the sums; the copy, where one is
// needed, at 4.5 TB/s.
struct PullCost { double plain, sliced; };
PullCost pull_cost(const maxk_graph* g, int dim, int k, int val_bytes, const void* dY, bool even_refused = false)
{
    const double N = (double)g->N, nnz = (double)g->nnz, row_bytes = (double)dim * val_bytes;
    const double miss = 1.0 - hot_share(g, 4e6 / row_bytes);
    int kp = 64;
    while (kp > 1 && kp / 2 >= k) kp /= 2;
    const double rounds = (double)std::min<int64_t>(g->chunk, g->max_in_degree) / (4.0 * (64 / kp));
    PullCost c;
    c.plain = 6e-6 + nnz * std::max(lines_touched(dim, k, val_bytes) * (5.0 + 12.0 * miss), 12.0 + 0.55 * k) * (k > 64 ? 1.15e-12 : 1e-12) +
              N * 200e-12 + 0.5 * rounds * 0.6e-6;
    const double slices = sliced_slices(dim, val_bytes), hit = hot_share(g, 24000.0);
    const bool in_place = sliced_in_place(dim, val_bytes);
    c.sliced = !sliced_supports(dY, g->N, dim, val_bytes) ||
                       (!in_place && !even_refused && is_refused(g, sliced_key(g, dim, val_bytes)) && sliced_copy_bytes(g->N, dim, val_bytes) > g->sliced_bytes)
                   ? HUGE_VAL
                   : 6e-6 + nnz * slices * (7e-12 * hit + 25e-12 * (1.0 - hit)) + N * slices * (60e-12 + 0.5e-12 * k) +
                         (in_place ? 0.0 : N * (row_bytes + slices * 128.0) / 4.5e12);
    return c;
}

// Backward kernel choice when the caller leaves it to the library: the lowest of five cost models, fitted on MI355X to
// 153 shapes (R-MAT and uniform graphs of 4 thousand to 1 million nodes, average degree 12 to 400; widths 64 to 512;
// k 8 to 128; fp32 and 16-bit dY) and the benchmark graphs.  Over those shapes the chosen kernel took 5 % longer than
// the best one on average with the kernels before pull by lane groups and tiles of 8 rows (profiles/backward_choice_over_shapes.txt; the largest misses, 2 times, are 16-bit dY on
// 60 k nodes of degree 240, where hub visits end the launches of slab pull later than the model has it).  The lines of expand/reduce
// and slab pull were fitted before product rows passed by L2 and long visits began a launch, and run high for both now: pull is
// taken on 42 k nodes, 3.3 M entries, k = 32 (243 us, expand/reduce 191), 40 k, 1.6 M, k = 32 (136 / 100), 118 k, 1.7 M, k = 64
// (241 / 208), 282 k, 3.4 M, k = 16 (247 / 214) and 169 k, 2.5 M, k = 32 (230 / 216; a whole pass 424 / 414).
// Times in seconds; `lines` = 128-byte lines of a dY row that an entry's k columns touch.
int auto_bwd_mode(const maxk_graph* g, int dim, int k, int val_bytes = 4, bool tiled_ok = true, bool even_refused = false, double* seconds = nullptr)
{
    const double N = (double)g->N, nnz = (double)g->nnz, row_bytes = (double)dim * val_bytes;
    const double lines = lines_touched(dim, k, val_bytes);

    const PullCost p = pull_cost(g, dim, k, val_bytes, nullptr, even_refused);
    const double pull = std::min(p.plain, p.sliced);

    // what was refused memory is out of the race until a reserve gets it (unless asked for the choice apart from that)
    const auto refused = [&](const RefusedKey& key) { return !even_refused && is_refused(g, key); };
    // expand/reduce: 8k bytes an entry through HBM, whatever the graph looks like (scalar stores when
    // k % 4 != 0, two-byte columns above dim 256)
    const double expand = nnz * k * 4.0 > 96e9 || (refused({kRefusedExpand, k}) && g->nnz * (int64_t)k > g->expand_floats) ? HUGE_VAL
                          : 8e-6 + nnz * (18e-12 + (dim > 256 ? 1.75e-12 : 1.5e-12) * k) * (k % 4 ? 1.7 : 1.0) +
                                N * (400e-12 + 0.22e-12 * row_bytes);

    // slab pull: lines from L2 at 5.2 ps (plus ~0.35 lines an entry of streamed arrays) and one launch a slab, ~22 us
    // with its ramp and tail
    const int32_t slab_rows = slab_rows_for(g, dim, val_bytes);
    const double n_slabs = std::ceil(N / slab_rows);
    const double slab = n_slabs * N >= 1.8e19 || refused({kRefusedSlab, slab_rows}) ? HUGE_VAL : 5e-6 + nnz * (lines + 0.35) * 5.2e-12 + n_slabs * 22e-6;

    // LDS-tiled: a (destination set, tile) step on each CU (the dim = 256 specialization is 3-5 times cheaper than the
    // general one), the entries, and fp32 atomics when the source rows are cut into ranges
    double tiled = HUGE_VAL;
    TiledShape sh;
    if (tiled_ok && val_bytes == 4 && tiled_shape(g->N, g->nnz, dim, k, sh) && !refused(tiled_key(sh, k))) {
        const double n_tiles = std::ceil(N / 16.0);  // (tiles of 8 where they are faster)
        if (sh.n_dsets * n_tiles < 2.6e8)
            tiled = 15e-6 + (dim == 256 ? 0.2e-6 : 0.5e-6 + 1.2e-9 * dim) * sh.n_dsets * n_tiles / 256.0 +
                    nnz * (3e-12 + 0.6e-12 * k) + (sh.R > 1 ? sh.R * N * k / 330e9 : 0.0);
        // It keeps one running sum an element and source range, pull and slab pull short ones.  On graphs of more than a few
        // thousand nodes it also has to win against slab pull by the models that were fitted on the dense and the
        // ogbn-proteins-like graph alone (within 10 % there; the ones above run high for slab pull where no hub ends its
        // launches), or it takes calls it is not faster for.  30 k nodes, width 256, k = 64, us (2-norm error against 64
        // bits) tiled / slab pull / pull: uniform, degree 300 405 (1.62e-7) / 395 (0.93e-7) / 693; degree 100 201 (1.01e-7)
        // / 193 / 219 (0.72e-7); R-MAT, degree 300 865 (4.9e-8) / 1074 / 584 (2.7e-8).
        if (sh.n_dsets * n_tiles >= 65536.0 &&
            1.05 * (150e-9 * sh.n_dsets * n_tiles / 256.0 + nnz * (3e-12 + 0.73e-12 * k)) >= nnz * (lines + 0.35) * 5.2e-12 + n_slabs * 10e-6)
            tiled = HUGE_VAL;
    }

    int mode = MAXK_BWD_PULL_CSC;
    double best = pull;
    if (1.05 * expand < best) { best = expand; mode = MAXK_BWD_EXPAND_REDUCE; }
    if (slab < best) { best = slab; mode = MAXK_BWD_SLAB_PULL; }
    if (tiled < best) { best = tiled; mode = MAXK_BWD_TILED; }
    if (seconds) *seconds = best;
    return mode;
}

// ---- the register-tiled kernel: how its sets are laid out, and where it stands in for the kernels above ----

// Rows that `sets` sets with a share x of the entries each use: a source of d entries is used by one with 1 - exp(-d x).
double regs_rows(const maxk_graph* g, double x)
{
    double rows = 0.0, before = 0.0;
    for (int i = 0; i < 33 && before < (double)g->N; ++i) {
        const double last = std::min((double)g->N, std::exp2(i)), count = last - before;
        const double entries = (g->hot_share[i] - (i ? g->hot_share[i - 1] : 0.f)) * (double)g->nnz;
        if (count > 0.0) rows += count * -std::expm1(-entries / count * x);
        before = last;
    }
    return rows;
}

// Seconds of a call with the sets of `sh`, the destinations behind its head by plain pull.  A step costs its entries (3.6 to 6.8
// ns each) and its rows: 0.63 us where they come from L2, 1.32 us more where each comes from beyond (even sets: an XCD's 32 CUs
// bring what one of them uses; by degree: 1.5 us), and the one hides a fifth of the other.  Fitted to 190 shapes of 1 k to 2.4 M
// nodes, degree 8 to 600: 8 % rms (even sets; 26 % before sums were added up with 16-byte loads), by degree 0.9 to 1.2 from 400 us up.
double regs_cost(const maxk_graph* g, const std::vector<std::pair<int32_t, int64_t>>& degrees, const RegsShape& sh, int dim, int val_bytes, int k)
{
    const double N = (double)g->N, nnz = (double)g->nnz, room = (double)regs_slots(sh.kr) * sh.groups * kRegsWaves * sh.spread;
    const double tile = regs_layout(sh.pitch).rows * kRegsWaves, rows_factor = sh.pitch > 1024 ? 1.15 : 1.0;
    const double b = sh.kr == 2 ? 6.8e-9 : sh.groups == 1 ? 4.6e-9 : sh.groups == 2 ? 3.55e-9 : 4.2e-9;
    const double hot = room * kRegsHotSlots / regs_slots(sh.kr);
    const bool even = sh.ranges > 0;
    int64_t shares = 0;
    for (const auto& [degree, n] : degrees) shares += n;
    double seconds = even ? 44e-6 : 180e-6, all_entries = 0.0, work = 0.0, copies = 0.0;
    auto run = degrees.begin();
    double nodes = run == degrees.end() ? 0.0 : (double)run->second, left = (double)sh.head;
    while (left > 0.0 && run != degrees.end()) {  // a run of `spread` sets at a time
        double in_run = std::min(room, left), at = 0.0, entries = 0.0;
        left -= in_run;
        bool cold = false;
        while (in_run > 0.0 && run != degrees.end()) {
            const double now = std::min(nodes, in_run), d = (double)run->first;
            entries += now * d;
            at += now;
            cold = cold || (at > hot && d > 0.0);
            in_run -= now;
            nodes -= now;
            if (nodes <= 0.0 && ++run != degrees.end()) nodes = (double)run->second;
        }
        all_entries += entries;
        const double used = regs_rows(g, entries / nnz / sh.spread), steps = sh.spread * std::max(1.0, used / tile) / 256.0;
        if (even) {
            const double p = std::min(1.0, used / N), missed = (1.0 - std::pow(1.0 - p, 32.0)) / (32.0 * std::max(p, 1e-9));
            const double run_work = b * entries / 256.0, run_copies = rows_factor * (0.63e-6 + 1.32e-6 * missed) * steps;
            seconds += std::max(run_work, run_copies) + 0.8 * std::min(run_work, run_copies);
            if (cold && sh.run) seconds += 10e-6;  // the sums that leave the registers are added up
        } else {
            work += 0.37e-6 * steps + b * entries / 256.0;
            copies += 1.5e-6 * steps * (sh.pitch > 1024 ? 1.5 : 1.0);
        }
    }
    seconds += std::max(work, copies) + 0.25 * std::min(work, copies);
    const double tail = nnz - all_entries, lines = lines_touched(dim, k, val_bytes), miss = 1.0 - hot_share(g, 4e6 / ((double)dim * val_bytes));
    if (shares > sh.head)
        seconds += 6e-6 + tail * std::max(lines * (5.0 + 12.0 * miss), 12.0 + 0.55 * k) * 1e-12 + (double)(shares - sh.head) * 200e-12;
    return seconds;
}

// Entries that a sum of the register-tiled kernel may take, so that it is no further off than the kernel `mode` that it stands in for
// (0: as many as it likes).  Plain pull of k > 32 adds up pieces of `chunk` entries four at a time; the others and the column slices
// a lane group's share of them; slab pull by rows takes eight at a time and then a sum per slab, which for the hubs that sets by
// degree hold is little.  The LDS-tiled kernel adds up a source range, slab pull's sampled form a destination, one by one
// whatever their number.  Errors go with the root of the length, and the mean length is a quarter to a half of the limit.  Error of
// the 12 largest destinations against 64 bits, k = 64, so / of the kernel before: 126 M entries on 2.4 M nodes 2.1e-7 / 4.3e-7 (plain pull);
// 41 M on 411 k, directed, mean weights 1.1e-7 / 1.5e-7 (column slices; 2.0e-7 with a limit of 512 here too).
int32_t regs_longest(const maxk_graph* g, int dim, int k, int val_bytes, int mode, bool sampled, bool even)
{
    if (mode == MAXK_BWD_TILED || sampled) return 0;
    const PullCost p = pull_cost(g, dim, k, val_bytes, nullptr, true);
    const bool sliced = g->pull_form == 0 ? p.sliced < p.plain : g->pull_form == 2 && p.sliced < HUGE_VAL;
    const int piece = std::min(g->chunk, 2048);
    if (mode == MAXK_BWD_SLAB_PULL && even) return std::max(128, piece / 8);
    return mode == MAXK_BWD_PULL_CSC && k > 32 && !sliced ? std::max(128, piece / 4) : 128;
}

// The layout for a shape (n_sets = 0: the other kernels are taken).  Even: as many sets as CUs (or fewer, in ranges of the rows),
// all sweeping the rows in step, so that an XCD brings a row into its L2 once.  By degree: as many sets as it takes.  Of the graph and
// the shape alone, whatever memory was refused: it is kept for the handle's life.
RegsShape best_regs_shape(const maxk_graph* g, int dim, int val_bytes, int k)
{
    RegsShape best, base;
    double seconds = HUGE_VAL, other = HUGE_VAL;
    const int mode = auto_bwd_mode(g, dim, k, val_bytes, true, true, &other);
    TiledShape tiled;
    (void)tiled_shape(g->N, g->nnz, dim, k, tiled);
    bool sampled = false;
    int32_t slab_run = 32;
    if (mode == MAXK_BWD_SLAB_PULL) {
        // Its line above was fitted where rows are long and degrees even.  Short rows cost their entries' instructions, few
        // entries a visit the visits, and a hub's visits end their launches late: us, the line above / measured, 31 M entries on
        // 96 k skewed nodes, width 128, bf16 539 / 3593; 39 M on 540 k, width 384 7515 / 11970; 27 M on 409 k, width 64, bf16 486 / 1456.
        // (The sampled form has fewer instructions an entry: 108 M on 371 k, width 128, k = 8, bf16 1954.)
        sampled = val_bytes == 4 ? 8 * k < dim : 16 * k <= dim;
        const double N = (double)g->N, nnz = (double)g->nnz, slabs = std::ceil(N / slab_rows_for(g, dim, val_bytes));
        const double visits = N * slabs * -std::expm1(-nnz / (N * slabs));
        const double entry = std::max((lines_touched(dim, k, val_bytes) + 0.35) * 4.3e-12, sampled ? 16e-12 : 27e-12);
        // Its sums: eight rows, those of a visit, one a slab.  One sum of as many entries and a tenth more is as far off, measured (14 M
        // entries on 34 k nodes, k = 46: with 25 / 28 / 32 entries 0.92 / 0.96 / 1.01 of its error).
        slab_run = (int32_t)std::clamp(1.1 * (8.0 + nnz / (8.0 * N * slabs) + slabs), 16.0, 32.0);
        other = std::max(0.85 * other, nnz * entry + visits * 45e-12 + slabs * 10e-6 + 15e-9 * (double)g->max_in_degree);
    }
    if (g->nnz > 0 && regs_fits(dim, val_bytes, k, base)) {
        const int64_t D = (int64_t)regs_slots(base.kr) * base.groups * kRegsWaves;
        const int32_t longest = regs_longest(g, dim, k, val_bytes, mode, sampled, true), hub_longest = regs_longest(g, dim, k, val_bytes, mode, sampled, false);
        // Even sets: a destination with many in-entries is several ones, or its wavefront's list holds up the others' at every
        // step and its sum gets long.  By degree few are: the sets that hold such ones are cut into units, and the entries
        // of one share rows (2.4 M nodes, k = 64: 8.0 ms with the even sets' line, 6.7 without one).
        using Degrees = std::vector<std::pair<int32_t, int64_t>>;
        const auto capped_at = [&](int64_t cap, Degrees& out) {
            int64_t shares = 0;
            for (const auto& [degree, n] : g->in_degrees) {
                const int64_t m = degree > cap ? (degree + cap - 1) / cap : 1;
                out.emplace_back((int32_t)(degree / m), n * m);
                shares += n * m;
            }
            std::stable_sort(out.begin(), out.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
            return shares;
        };
        const int64_t cap = std::max<int64_t>(64, std::min(8 * (g->nnz / g->N + 1), g->nnz / 16384)), hub_cap = hub_longest ? 64ll * hub_longest : g->nnz;
        Degrees capped, hubs_capped;
        const int64_t capped_shares = capped_at(cap, capped), hubs_capped_shares = capped_at(hub_cap, hubs_capped);
        const auto consider = [&](int64_t sets, int64_t spread, int32_t ranges) {
            RegsShape sh = base;
            const Degrees& degrees = ranges ? capped : hubs_capped;
            const int64_t shares = ranges ? capped_shares : hubs_capped_shares;
            sh.cap = ranges ? cap : hub_cap;
            sh.n_sets = (int32_t)sets;
            sh.spread = (int32_t)spread;
            sh.ranges = ranges;
            sh.longest = ranges ? longest : hub_longest;
            sh.head = std::min<int64_t>(shares, sets * D);
            // Pull and expand/reduce: 12, or 8 where a sum of 12 is most of many results, because most destinations have few entries and
            // sets of one range hold them (15 M entries on 989 k nodes, k = 32: error 4.35e-8 before, 4.59e-8 with 12, 4.29e-8 with 8).
            const bool few = g->nnz < 24 * g->N && ranges <= 1 && 2 * sh.head > shares;
            sh.run = mode == MAXK_BWD_SLAB_PULL ? slab_run : mode != MAXK_BWD_TILED ? (few ? 8 : 12) : ranges >= tiled.R ? 0 : 64;
            // the tail is the end of the pull's item list: none of its destinations may be several or split there
            int64_t above = 0;
            for (const auto& [degree, n] : degrees) {
                if (degree < std::min<int64_t>(g->chunk, sh.cap) / 2) break;
                above += n;
            }
            if (sh.head < shares && sh.head < above && g->max_in_degree >= std::min<int64_t>(g->chunk, sh.cap) / 2) return;
            const double t = regs_cost(g, degrees, sh, dim, val_bytes, k);
            if (t < seconds) { seconds = t; best = sh; }
        };
        for (int R = 1; R <= 8 && g->bwd_regs != 3; R *= 2) consider(256 / R, 256 / R, R);
        for (int64_t rounds = 2; rounds <= 8 && g->bwd_regs != 3 && (rounds - 1) * 256 * D < capped_shares; ++rounds) consider(256 * rounds, 256, 1);
        int64_t nodes = 0;
        int next = 128;
        for (const auto& [degree, n] : hubs_capped) {
            while (nodes > 0 && degree < next && next >= 4) {
                consider((nodes + D - 1) / D, 1, 0);
                next /= 2;
            }
            nodes += n;
        }
        if (g->bwd_regs == 3) consider((nodes + D - 1) / D, 1, 0);
    }
    // The others' lines over what was measured on 190 shapes: slab pull 0.45 to 1.3, mostly below 1; pull and tiled 0.9 to 1.2;
    // expand/reduce 1.0 to 1.2, but 1.2 to 1.6 where dY stays in the 256 MB Infinity Cache.  This kernel's: 0.75 to 1.25.
    // Against pull, this kernel's runs low where rows are short (256 bytes and k > 32: 1.2 to 1.45; k > 16: 1.2 to 1.3 where a
    // graph's frequent sources, which pull finds in L2, hold much of its entries; 512 and k > 64: 1.2 to 1.45).
    const double pull_line = base.pitch == 256 && k > 32 ? 0.7 : base.pitch == 256 && k > 16 && hot_share(g, 16384.0) > 0.4 ? 0.72
                             : k <= 64 ? 1.0 : best.run == 8 ? 0.8 : base.pitch > 512 ? 0.87 : best.ranges ? 0.83 : 0.7;
    const bool small = other < 600e-6;
    const double line = mode == MAXK_BWD_SLAB_PULL ? (small ? 0.9 : 1.0)
                        : mode == MAXK_BWD_EXPAND_REDUCE ? ((double)g->N * dim * val_bytes > 256e6 ? 0.85 : 0.7)
                        : mode == MAXK_BWD_PULL_CSC ? std::min(small ? 0.8 : 0.9, pull_line) : (small ? 0.8 : 0.9);
    if (g->bwd_regs < 2 && !(seconds < line * other)) best = RegsShape();
    return best;
}

RegsShape regs_choice(maxk_graph* g, int dim, int val_bytes, int k)
{
    if (g->bwd_regs == 1) return RegsShape();
    for (const auto& c : g->regs_choices)
        if (c.dim == dim && c.val_bytes == val_bytes && c.k == k) return c.shape;
    try {
        const RegsShape best = best_regs_shape(g, dim, val_bytes, k);
        g->regs_choices.push_back({dim, val_bytes, k, best});
        return best;
    } catch (const std::bad_alloc&) {  // the other kernels, and it is worked out again
        return RegsShape();
    }
}

// The backward kernel of a call and the tables it walks, which are built where they are missing.
struct BwdPlan {
    int mode = MAXK_BWD_PULL_CSC;
    bool sliced = false;  // the pull's column-sliced form
    TiledSet* T = nullptr;
    RegsSet* M = nullptr;  // the register-tiled kernel stands in for `mode`
    SlabSet* S = nullptr;
};

// Chooses the kernel and builds what it lacks, for a reserve (stream = nullptr) and for a compute call alike.  The
// library's own choice goes on to the next best kernel when memory runs out, down to plain pull, which needs no buffer of
// its own; while the call is being captured nothing may be allocated, and plain pull stands in for what is missing.
maxk_status plan_bwd(maxk_graph* g, int dim, int k, int vb, bool tiled_ok, const void* dY, const hipStream_t* stream, BwdPlan& plan)
{
    const bool automatic = g->bwd_mode == MAXK_BWD_AUTO;
    const auto captured = [&] { return stream && capturing(*stream); };
    const auto existing_only = [&] { return automatic && captured(); };
    if (automatic && aligned(dY, 16)) {
        const RegsShape sh = regs_choice(g, dim, vb, k);
        if (sh.n_sets && !regs_refused(g, sh)) {
            const maxk_status st = regs_for(g, sh, captured, &plan.M);
            if (st == MAXK_OK || st == MAXK_HIP_ERROR) return st;
        }
    }
    int mode = automatic ? auto_bwd_mode(g, dim, k, vb, tiled_ok) : g->bwd_mode;
    for (;;) {
        maxk_status st = MAXK_OK;
        plan = BwdPlan();
        plan.mode = mode;
        if (mode == MAXK_BWD_TILED) {
            st = tiled_ok ? tiled_for(g, dim, k, existing_only, &plan.T) : MAXK_UNSUPPORTED;
            if (st == MAXK_UNSUPPORTED) plan.mode = MAXK_BWD_SLAB_PULL;  // shapes, formats and alignments the tiled kernel does not take
        }
        if (plan.mode == MAXK_BWD_SLAB_PULL) st = slabs_for(g, slab_rows_for(g, dim, vb), existing_only, &plan.S);
        if (mode == MAXK_BWD_EXPAND_REDUCE) {
            st = g->nnz * (int64_t)k > g->expand_floats && existing_only() ? MAXK_OUT_OF_MEMORY : ensure_expand(g, k);
        }
        if (mode == MAXK_BWD_PULL_CSC) {
            const PullCost p = pull_cost(g, dim, k, vb, dY);
            plan.sliced = g->pull_form == 0 ? p.sliced < p.plain : g->pull_form == 2 && p.sliced < HUGE_VAL;
            if (plan.sliced && !sliced_in_place(dim, vb)) {
                st = sliced_copy_bytes(g->N, dim, vb) > g->sliced_bytes && captured() ? MAXK_OUT_OF_MEMORY : ensure_sliced(g, dim, vb);
                if (st == MAXK_OUT_OF_MEMORY) {
                    plan.sliced = false;
                    st = MAXK_OK;
                }
            }
        }
        if (st != MAXK_OUT_OF_MEMORY || !automatic) return st;
        const int next = auto_bwd_mode(g, dim, k, vb, tiled_ok);
        mode = next == mode ? MAXK_BWD_PULL_CSC : next;  // (the same again: nothing was refused, the call is being captured)
    }
}

maxk_status reserve_shape(maxk_graph* g, int dim, int k, int dy_value_type)
{
    maxk_status st = ensure_workspace(g, dim, k);
    if (st != MAXK_OK) return st;
    if (const int per_bin = sweep_rows(g, dim, k, dim <= 256 ? 1 : 2, 4)) {  // (narrower records may not need it)
        SweepSet* W = nullptr;
        forget_refused(g, {kRefusedSweep, sweep_groups(k), sweep_batch(k), per_bin});
        (void)sweep_for(g, k, dim, per_bin, false, &W);  // (not built: row by row)
    }
    int largest[3] = {0, 0, 0}, bytes = 0;  // k', index and value bytes of the largest repacked record among k' <= k
    for (int vb = 2; vb <= 4; vb += 2) {
        for (int ib = 1; ib <= 4; ib *= 2) {
            for (int kk = 1; kk <= k && kk * (vb + ib) <= std::max(96, g->fwd_pack_max); ++kk) {
                if (!fwd_uses_packed(g, kk, ib, vb) || fwd_packed_record_bytes(kk, ib, vb) <= bytes) continue;
                bytes = fwd_packed_record_bytes(kk, ib, vb);
                largest[0] = kk, largest[1] = ib, largest[2] = vb;
            }
        }
    }
    if (bytes) {
        st = ensure_packed(g, largest[0], largest[1], largest[2]);
        if (st != MAXK_OK) return st;
    }
    const int vb = value_bytes(dy_value_type);
    forget_refused(g, {kRefusedExpand, k});
    forget_refused(g, {kRefusedSlab, slab_rows_for(g, dim, vb)});
    forget_refused(g, sliced_key(g, dim, vb));
    TiledShape sh;
    if (tiled_shape(g->N, g->nnz, dim, k, sh)) forget_refused(g, tiled_key(sh, k));
    if (const RegsShape rs = regs_choice(g, dim, vb, k); rs.n_sets) std::erase(g->regs_refused, rs);
    BwdPlan plan;
    return g->nnz ? plan_bwd(g, dim, k, vb, true, nullptr, nullptr, plan) : MAXK_OK;
}

bool bad_index_bytes(int index_bytes, int dim)
{
    if (index_bytes == 1) return dim > 256;
    if (index_bytes == 2) return dim > 65536;
    return index_bytes != 4;
}

}  // namespace
}  // namespace maxk

using namespace maxk;

extern "C" {

MAXK_API maxk_status maxk_graph_create(maxk_graph** out, int64_t N, int64_t nnz, const int32_t* d_rowptr,
                              const int32_t* d_colidx, const float* d_val, void* stream)
{
    if (!out) return MAXK_INVALID_ARGUMENT;
    *out = nullptr;
    if (N < 0 || nnz < 0 || N > 0x7FFFFFF0ll || nnz > 0x7FFFFFF0ll) return MAXK_INVALID_ARGUMENT;
    if (!d_rowptr || (nnz > 0 && (!d_colidx || !d_val))) return MAXK_INVALID_ARGUMENT;
    if (!aligned(d_rowptr, 4) || !aligned(d_colidx, 4) || !aligned(d_val, 4)) return MAXK_INVALID_ARGUMENT;
    hipStream_t s = (hipStream_t)stream;

    maxk_graph* g = new (std::nothrow) maxk_graph();
    if (!g) return MAXK_OUT_OF_MEMORY;
    g->N = N;
    g->nnz = nnz;
    g->d_rowptr = d_rowptr;
    g->d_col = d_colidx;
    g->d_val = d_val;
    g->chunk = env_int("MAXK_CHUNK", default_chunk(nnz), 64, 1 << 20);
    g->slab_kb = env_int("MAXK_SLAB_KB", 3584, 64, 1 << 20);
    g->fwd_pack_max = env_int("MAXK_FWD_PACK_MAX", -1, -1, 1 << 20);
    g->fwd_sweep = env_int("MAXK_FWD_SWEEP", 0, 0, 2);
    g->pull_form = env_int("MAXK_PULL_FORM", 0, 0, 2);
    g->bwd_regs = env_int("MAXK_BWD_REGS", 0, 0, 3);
    (void)hipGetDevice(&g->device);
    {
        const maxk_status sst = noalloc_scratch_address(&g->d_noalloc_scratch);
        if (sst != MAXK_OK) { delete g; return sst; }
    }

    maxk_status st = MAXK_OK;
    try {
        std::vector<int32_t> h_rowptr((size_t)N + 1);
        hipError_t e = hipMemcpyAsync(h_rowptr.data(), d_rowptr, sizeof(int32_t) * (size_t)(N + 1), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) { st = hip_fail(e); goto fail; }
        if (h_rowptr[0] != 0 || (int64_t)h_rowptr[(size_t)N] != nnz) { st = MAXK_INVALID_ARGUMENT; goto fail; }
        for (int64_t i = 0; i < N; ++i)
            if (h_rowptr[(size_t)i + 1] < h_rowptr[(size_t)i]) { st = MAXK_INVALID_ARGUMENT; goto fail; }

        std::vector<WorkItem> items;
        std::vector<SplitRow> split;
        int64_t n_slots = 0, max_len = 0;
        build_items(h_rowptr, N, g->chunk, items, split, n_slots, max_len);
        g->max_degree = max_len;
        for (const WorkItem& w : items) {
            const int32_t len = w.end - w.begin;
            if (g->csr_lengths.empty() || g->csr_lengths.back().first != len) g->csr_lengths.emplace_back(len, 0);
            ++g->csr_lengths.back().second;
        }
        hot_source_shares(h_rowptr, N, nnz, g->hot_share);
        st = upload_items(items, split, n_slots, g->csr_items, s);
        if (st != MAXK_OK) goto fail;

        std::vector<int32_t> h_csc_ptr;
        st = build_csc(g, h_csc_ptr, s);
        if (st != MAXK_OK) goto fail;
        build_items(h_csc_ptr, N, g->chunk, items, split, n_slots, max_len);
        g->max_in_degree = max_len;
        count_lengths(h_csc_ptr, items, split, g->in_degrees);
        st = upload_items(items, split, n_slots, g->csc_items, s);
        if (st != MAXK_OK) goto fail;
    } catch (const std::bad_alloc&) {
        st = MAXK_OUT_OF_MEMORY;
        goto fail;
    }
    short_item_workspace(g);
    *out = g;
    return MAXK_OK;
fail:
    maxk_graph_destroy(g);
    return st;
}

MAXK_API maxk_status maxk_graph_destroy(maxk_graph* g)
{
    if (!g) return MAXK_OK;
    (void)hipFree(g->csr_items.d_items);
    (void)hipFree(g->csr_items.d_split);
    (void)hipFree(g->csc_items.d_items);
    (void)hipFree(g->csc_items.d_split);
    (void)hipFree(g->d_csc_ptr);
    (void)hipFree(g->d_csc_src);
    (void)hipFree(g->d_csc_val);
    (void)hipFree(g->d_csc_entry);
    (void)hipFree(g->d_expand);
    (void)hipFree(g->d_packed);
    (void)hipFree(g->d_sliced);
    for (char* p : g->sliced_before) (void)hipFree(p);
    for (SlabSet* S : g->slab_cache) { free_slabs(*S); delete S; }
    for (TiledSet* T : g->tiled_cache) { free_tiled(*T); delete T; }
    for (RegsSet* T : g->regs_cache) { free_regs(*T); delete T; }
    for (SweepSet* W : g->sweep_cache) { free_sweep(*W); delete W; }
    (void)hipFree(g->d_partials);
    delete g;
    return MAXK_OK;
}

MAXK_API maxk_status maxk_graph_reserve_narrow(maxk_graph* g, int32_t dim, int32_t k, int32_t dy_value_type)
{
    if (!g || dim < 1 || k < 1 || k > dim) return MAXK_INVALID_ARGUMENT;
    if (dy_value_type < MAXK_VALUE_F32 || dy_value_type > MAXK_VALUE_F16) return MAXK_INVALID_ARGUMENT;
    if (dim > MAXK_MAX_DIM) return MAXK_UNSUPPORTED;
    if (g->N == 0) return MAXK_OK;
    const maxk_status st = reserve_shape(g, dim, k, dy_value_type);
    return st == MAXK_OK ? note_reserved(g, dim, k) : st;
}

MAXK_API maxk_status maxk_graph_reserve(maxk_graph* g, int32_t dim, int32_t k)
{
    return maxk_graph_reserve_narrow(g, dim, k, MAXK_VALUE_F32);
}

MAXK_API maxk_status maxk_graph_set_bwd_mode(maxk_graph* g, int32_t mode)
{
    if (!g || mode < MAXK_BWD_AUTO || mode > MAXK_BWD_TILED) return MAXK_INVALID_ARGUMENT;
    g->bwd_mode = mode;
    return MAXK_OK;
}

MAXK_API int32_t maxk_graph_bwd_choice(const maxk_graph* g, int32_t dim, int32_t k)
{
    if (!g || dim < 1 || k < 1 || k > dim) return MAXK_INVALID_ARGUMENT;
    return g->bwd_mode == MAXK_BWD_AUTO ? auto_bwd_mode(g, dim, k) : g->bwd_mode;
}

MAXK_API maxk_status maxk_graph_info(const maxk_graph* g, int64_t* N, int64_t* nnz, int64_t* n_fwd_items, int64_t* n_split_rows,
                            int64_t* max_degree, int64_t* workspace_bytes)
{
    if (!g) return MAXK_INVALID_ARGUMENT;
    if (N) *N = g->N;
    if (nnz) *nnz = g->nnz;
    if (n_fwd_items) *n_fwd_items = g->csr_items.n_items;
    if (n_split_rows) *n_split_rows = g->csr_items.n_split;
    if (max_degree) *max_degree = g->max_degree;
    if (workspace_bytes)
    {
        int64_t regs = 0;
        for (const RegsSet* T : g->regs_cache) regs += (T->part_floats + T->extra_floats) * (int64_t)sizeof(float);
        *workspace_bytes = regs + (g->partial_floats + g->expand_floats) * (int64_t)sizeof(float) + g->packed_bytes + g->sliced_bytes +
                           g->sliced_before_bytes;
    }
    return MAXK_OK;
}

MAXK_API maxk_status maxk_topk_cbsr_narrow(const float* d_H, int64_t N, int32_t dim, int32_t k, void* d_sp_data,
                                           int32_t value_type, void* d_sp_index, int32_t index_bytes, void* stream)
{
    if (N < 0 || dim < 1 || k < 1 || k > dim || bad_index_bytes(index_bytes, dim)) return MAXK_INVALID_ARGUMENT;
    if (value_type < MAXK_VALUE_F32 || value_type > MAXK_VALUE_F16) return MAXK_INVALID_ARGUMENT;
    if (dim > MAXK_MAX_DIM) return MAXK_UNSUPPORTED;
    if (N > 0x7FFFFFF0ll) return MAXK_INVALID_ARGUMENT;
    if (N == 0) return MAXK_OK;
    if (!d_H || !d_sp_data || !d_sp_index) return MAXK_INVALID_ARGUMENT;
    if (!aligned(d_H, 4) || !aligned(d_sp_data, (size_t)value_bytes(value_type)) ||
        !aligned(d_sp_index, (size_t)index_bytes))
        return MAXK_INVALID_ARGUMENT;
    return launch_topk(d_H, N, dim, k, d_sp_data, value_type, d_sp_index, index_bytes, (hipStream_t)stream);
}

MAXK_API maxk_status maxk_topk_cbsr(const float* d_H, int64_t N, int32_t dim, int32_t k, float* d_sp_data, void* d_sp_index,
                           int32_t index_bytes, void* stream)
{
    return maxk_topk_cbsr_narrow(d_H, N, dim, k, d_sp_data, MAXK_VALUE_F32, d_sp_index, index_bytes, stream);
}

MAXK_API maxk_status maxk_spgemm_fwd_narrow(maxk_graph* g, const void* d_sp_data, int32_t value_type,
                                            const void* d_sp_index, int32_t index_bytes, int32_t dim, int32_t k,
                                            float* d_Y, void* stream)
{
    if (!g || dim < 1 || k < 1 || k > dim || bad_index_bytes(index_bytes, dim)) return MAXK_INVALID_ARGUMENT;
    if (value_type < MAXK_VALUE_F32 || value_type > MAXK_VALUE_F16) return MAXK_INVALID_ARGUMENT;
    if (dim > MAXK_MAX_DIM) return MAXK_UNSUPPORTED;
    if (g->N == 0) return MAXK_OK;
    if (!d_sp_data || !d_sp_index || !d_Y) return MAXK_INVALID_ARGUMENT;
    const int vb = value_bytes(value_type);
    if (!aligned(d_sp_data, (size_t)vb) || !aligned(d_Y, 4) || !aligned(d_sp_index, (size_t)index_bytes))
        return MAXK_INVALID_ARGUMENT;
    maxk_status st = ensure_workspace(g, dim, k);
    if (st != MAXK_OK) return st;
    char* packed = nullptr;
    if (fwd_uses_packed(g, k, index_bytes, vb)) {
        st = ensure_packed(g, k, index_bytes, vb);
        if (st != MAXK_OK) return st;
        packed = g->d_packed;
    }
    if (const int per_bin = sweep_rows(g, dim, k, index_bytes, vb)) {
        SweepSet* W = nullptr;
        st = sweep_for(g, k, dim, per_bin, reserved_for(g, dim, k) || capturing((hipStream_t)stream), &W);
        if (st == MAXK_OK)
            return launch_spgemm_fwd_sweep(g->csr_items, *W, d_sp_data, value_type, d_sp_index, index_bytes, g->N, packed, dim, k,
                                           d_Y, g->d_partials, (hipStream_t)stream);
    }
    return launch_spgemm_fwd(g->csr_items, g->d_col, g->d_val, d_sp_data, value_type, d_sp_index, index_bytes, g->N, packed,
                             dim, k, d_Y, g->d_partials, (hipStream_t)stream);
}

MAXK_API maxk_status maxk_spgemm_fwd(maxk_graph* g, const float* d_sp_data, const void* d_sp_index, int32_t index_bytes,
                            int32_t dim, int32_t k, float* d_Y, void* stream)
{
    return maxk_spgemm_fwd_narrow(g, d_sp_data, MAXK_VALUE_F32, d_sp_index, index_bytes, dim, k, d_Y, stream);
}

MAXK_API maxk_status maxk_spgemm_fwd_noalloc(maxk_graph* g, const float* d_sp_data, const void* d_sp_index,
                                             int32_t index_bytes, int32_t dim, int32_t k, float* d_Y, void* stream)
{
    if (!g || dim < 1 || k < 1 || k > dim || bad_index_bytes(index_bytes, dim)) return MAXK_INVALID_ARGUMENT;
    if (dim > MAXK_MAX_DIM) return MAXK_UNSUPPORTED;
    if (g->N == 0) return MAXK_OK;
    if (!d_sp_data || !d_sp_index || !d_Y) return MAXK_INVALID_ARGUMENT;
    if (!aligned(d_sp_data, 4) || !aligned(d_Y, 4) || !aligned(d_sp_index, (size_t)index_bytes)) return MAXK_INVALID_ARGUMENT;
    int device = -1;
    MAXK_HIP_TRY(hipGetDevice(&device));
    if (device != g->device || !g->d_noalloc_scratch) return MAXK_INVALID_ARGUMENT;  // the array is per GPU
    // layout of the scratch array: [partial rows of split rows | repacked CBSR, if it fits]
    const int64_t partial_bytes = (g->csr_items.n_slots * (int64_t)dim * 4 + 255) & ~(int64_t)255;
    if (partial_bytes > (int64_t)MAXK_NOALLOC_SCRATCH_BYTES) return MAXK_SCRATCH_TOO_SMALL;
    float* partials = reinterpret_cast<float*>(g->d_noalloc_scratch);
    char* packed = nullptr;
    if (fwd_uses_packed(g, k, index_bytes, 4) &&
        partial_bytes + g->N * (int64_t)fwd_packed_record_bytes(k, index_bytes, 4) <= (int64_t)MAXK_NOALLOC_SCRATCH_BYTES)
        packed = reinterpret_cast<char*>(g->d_noalloc_scratch) + partial_bytes;
    // nothing in the array has to start at zero: the kernels write every partial row and every record they read
    if (const int per_bin = sweep_rows(g, dim, k, index_bytes, 4)) {  // where the regrouped A is there already
        SweepSet* W = nullptr;
        if (sweep_for(g, k, dim, per_bin, true, &W) == MAXK_OK)
            return launch_spgemm_fwd_sweep(g->csr_items, *W, d_sp_data, MAXK_VALUE_F32, d_sp_index, index_bytes, g->N, packed, dim,
                                           k, d_Y, partials, (hipStream_t)stream);
    }
    return launch_spgemm_fwd(g->csr_items, g->d_col, g->d_val, d_sp_data, MAXK_VALUE_F32, d_sp_index, index_bytes, g->N,
                             packed, dim, k, d_Y, partials, (hipStream_t)stream);
}

MAXK_API maxk_status maxk_sspmm_bwd_narrow(maxk_graph* g, const void* d_dY, int32_t value_type, const void* d_sp_index,
                                           int32_t index_bytes, int32_t dim, int32_t k, float* d_dXs, void* stream)
{
    if (!g || dim < 1 || k < 1 || k > dim || bad_index_bytes(index_bytes, dim)) return MAXK_INVALID_ARGUMENT;
    if (value_type < MAXK_VALUE_F32 || value_type > MAXK_VALUE_F16) return MAXK_INVALID_ARGUMENT;
    if (dim > MAXK_MAX_DIM) return MAXK_UNSUPPORTED;
    if (g->N == 0) return MAXK_OK;
    if (!d_dY || !d_sp_index || !d_dXs) return MAXK_INVALID_ARGUMENT;
    const int vb = value_bytes(value_type);
    if (!aligned(d_dY, (size_t)vb) || !aligned(d_dXs, 4) || !aligned(d_sp_index, (size_t)index_bytes))
        return MAXK_INVALID_ARGUMENT;
    maxk_status st = ensure_workspace(g, dim, k);
    if (st != MAXK_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    if (g->nnz == 0) return launch_fill_zero(d_dXs, g->N * (int64_t)k, s);
    BwdPlan plan;
    st = plan_bwd(g, dim, k, vb, tiled_supports(d_dY, value_type, d_sp_index, index_bytes, dim, k), d_dY, &s, plan);
    if (st != MAXK_OK) return st;
    if (plan.M) {
        st = launch_bwd_regs(*plan.M, d_dY, value_type, d_sp_index, index_bytes, g->N, dim, k, d_dXs, s);
        const int64_t tail = plan.M->n_tail;
        if (st != MAXK_OK || tail <= 0) return st;
        ItemList rest = g->csc_items;
        rest.d_items += rest.n_items - tail;
        rest.n_items = tail;
        rest.n_split = rest.n_slots = 0;
        return launch_bwd_pull(rest, g->d_csc_src, g->d_csc_val, d_dY, value_type, d_sp_index, index_bytes, g->N, dim, k, pull_tail_by_units(g, dim, k, vb), d_dXs,
                               g->d_partials, s);
    }
    if (plan.mode == MAXK_BWD_TILED)
        return launch_bwd_tiled(*plan.T, d_dY, value_type, d_sp_index, index_bytes, g->N, dim, k, d_dXs, s);
    if (plan.mode == MAXK_BWD_SLAB_PULL)
        return launch_bwd_slab_pull(*plan.S, d_dY, value_type, d_sp_index, index_bytes, g->N, dim, k, d_dXs, s);
    if (plan.mode == MAXK_BWD_EXPAND_REDUCE)
        return launch_bwd_expand_reduce(g->csr_items, g->d_col, g->d_val, g->csc_items, g->d_csc_entry, d_dY, value_type,
                                        d_sp_index, index_bytes, dim, k, products_past_l2(g->N, g->nnz, dim, k, index_bytes, vb),
                                        g->d_expand, d_dXs, g->d_partials, s);
    if (plan.mode == MAXK_BWD_PULL_CSC) {
        if (plan.sliced) {
            st = launch_bwd_sliced(g->csc_items, g->d_csc_src, g->d_csc_val, d_dY, value_type, d_sp_index, index_bytes, g->N, dim, k,
                                   sliced_in_place(dim, vb) ? nullptr : g->d_sliced, d_dXs, g->d_partials, s);
            if (st != MAXK_UNSUPPORTED) return st;
        }
        return launch_bwd_pull(g->csc_items, g->d_csc_src, g->d_csc_val, d_dY, value_type, d_sp_index, index_bytes, g->N, dim, k,
                               pull_by_units(g, dim, k, vb), d_dXs, g->d_partials, s);
    }
    return launch_bwd_push(g->csr_items, g->d_col, g->d_val, d_dY, value_type, d_sp_index, index_bytes, g->N, dim, k, d_dXs, s);
}

MAXK_API maxk_status maxk_sspmm_bwd(maxk_graph* g, const float* d_dY, const void* d_sp_index, int32_t index_bytes, int32_t dim,
                           int32_t k, float* d_dXs, void* stream)
{
    return maxk_sspmm_bwd_narrow(g, d_dY, MAXK_VALUE_F32, d_sp_index, index_bytes, dim, k, d_dXs, stream);
}

MAXK_API maxk_status maxk_cbsr_scatter(const float* d_values, const void* d_sp_index, int32_t index_bytes, int64_t N,
                                       int32_t dim, int32_t k, float* d_dense, void* stream)
{
    if (N < 0 || dim < 1 || k < 1 || k > dim || bad_index_bytes(index_bytes, dim)) return MAXK_INVALID_ARGUMENT;
    if (dim > MAXK_MAX_DIM) return MAXK_UNSUPPORTED;
    if (N > 0x7FFFFFF0ll) return MAXK_INVALID_ARGUMENT;
    if (N == 0) return MAXK_OK;
    if (!d_values || !d_sp_index || !d_dense) return MAXK_INVALID_ARGUMENT;
    if (!aligned(d_values, 4) || !aligned(d_dense, 4) || !aligned(d_sp_index, (size_t)index_bytes))
        return MAXK_INVALID_ARGUMENT;
    return launch_cbsr_scatter(d_values, d_sp_index, index_bytes, N, dim, k, d_dense, (hipStream_t)stream);
}

MAXK_API maxk_status spmm_baseline(maxk_graph* g, const float* d_H, int32_t dim, float* d_Y, void* stream)
{
    if (!g || dim < 1) return MAXK_INVALID_ARGUMENT;
    if (dim > MAXK_MAX_DIM) return MAXK_UNSUPPORTED;
    if (g->N == 0) return MAXK_OK;
    if (!d_H || !d_Y || !aligned(d_H, 4) || !aligned(d_Y, 4)) return MAXK_INVALID_ARGUMENT;
    maxk_status st = ensure_workspace(g, dim, 1);
    if (st != MAXK_OK) return st;
    return launch_spmm(g->csr_items, g->d_col, g->d_val, d_H, dim, d_Y, g->d_partials, (hipStream_t)stream);
}

MAXK_API const char* maxk_status_string(maxk_status s)
{
    switch (s) {
        case MAXK_OK: return "ok";
        case MAXK_INVALID_ARGUMENT: return "invalid argument";
        case MAXK_UNSUPPORTED: return "unsupported size";
        case MAXK_HIP_ERROR: return "HIP runtime error";
        case MAXK_OUT_OF_MEMORY: return "out of device or host memory";
        case MAXK_SCRATCH_TOO_SMALL: return "the input needs more scratch memory than the library's fixed array holds";
        default: return "unknown status";
    }
}

MAXK_API int32_t maxk_fwd_private_copies(int32_t k) { return k < 1 ? MAXK_INVALID_ARGUMENT : fwd_private_copies(k); }

MAXK_API int32_t maxk_expand_past_l2(int64_t N, int64_t nnz, int32_t dim, int32_t k, int32_t index_bytes, int32_t dy_value_type)
{
    return products_past_l2(N, nnz, dim, k, index_bytes, value_bytes(dy_value_type));
}

MAXK_API int32_t maxk_scatter_past_l2(int64_t N, int32_t dim) { return scatter_past_l2(N, dim); }

MAXK_API maxk_status maxk_graph_cached_tables(const maxk_graph* g, int32_t* n_slab_tables, int32_t* n_tiled_tables)
{
    if (!g) return MAXK_INVALID_ARGUMENT;
    if (n_slab_tables) *n_slab_tables = (int32_t)g->slab_cache.size();
    if (n_tiled_tables) *n_tiled_tables = (int32_t)g->tiled_cache.size();
    return MAXK_OK;
}

MAXK_API int32_t maxk_lone_visit_line(int32_t longest, int64_t entries) { return lone_visit_line(longest, entries); }

MAXK_API int32_t maxk_graph_regs_stands_in(maxk_graph* g, int32_t dim, int32_t k, int32_t dy_value_type)
{
    if (!g || dim < 1 || k < 1 || k > dim || dy_value_type < MAXK_VALUE_F32 || dy_value_type > MAXK_VALUE_F16) return MAXK_INVALID_ARGUMENT;
    if (g->bwd_mode != MAXK_BWD_AUTO || g->nnz == 0) return 0;
    const RegsShape sh = regs_choice(g, dim, value_bytes(dy_value_type), k);
    return sh.n_sets && !regs_refused(g, sh);
}

MAXK_API int32_t maxk_graph_regs_tables(const maxk_graph* g) { return g ? (int32_t)g->regs_cache.size() : MAXK_INVALID_ARGUMENT; }

MAXK_API maxk_status maxk_regs_step_list(uint32_t record0, uint32_t records, uint32_t step, uint32_t* first, uint32_t* copied)
{
    if (!first || !copied) return MAXK_INVALID_ARGUMENT;
    const RegsStepList list = regs_step_list(record0, records, step);
    *first = list.first;
    *copied = regs_copied(list.records);
    return MAXK_OK;
}

MAXK_API int32_t maxk_fwd_by_units(int32_t k, int32_t dim, int32_t value_type, int64_t items, int64_t entries)
{
    return k < 1 ? MAXK_INVALID_ARGUMENT : fwd_by_units(k, dim, value_bytes(value_type), items, entries);
}

MAXK_API int32_t maxk_pull_by_units(int32_t dim, int32_t k, int32_t value_type, int64_t N, int64_t nnz, double beyond)
{
    return k < 1 || dim < k ? MAXK_INVALID_ARGUMENT : pull_by_units(dim, k, value_bytes(value_type), N, nnz, beyond);
}

MAXK_API int64_t maxk_entry_batch(uint32_t base, uint32_t ahead, uint32_t end) { return batch_begin(base + ahead, end); }

MAXK_API int64_t maxk_graph_regs_table(const maxk_graph* g, int32_t i, int32_t which, void* out, int64_t bytes)
{
    if (!g || i < 0 || (size_t)i >= g->regs_cache.size()) return MAXK_INVALID_ARGUMENT;
    const RegsSet& T = *g->regs_cache[(size_t)i];
    const RegsShape& sh = T.shape;
    const RegsLayout layout = regs_layout(sh.pitch);
    const int64_t slots = regs_slots(sh.kr), accumulators = (int64_t)sh.n_sets * kRegsWaves * slots * sh.groups;
    const int64_t sizes[] = {sh.pitch, sh.groups, sh.kr, sh.n_sets, sh.spread, sh.ranges, sh.run, sh.longest, sh.cap, sh.head, slots, layout.rows, layout.head,
                             T.n_steps, T.n_records, T.n_units, T.n_parts, T.n_sums, T.n_split, T.n_tail, T.part_floats, T.hot_parts,
                             T.extra_floats};
    const std::pair<const void*, int64_t> tables[] = {
        {nullptr, (int64_t)sizeof(sizes)},
        {T.d_rec, T.n_records * (int64_t)sizeof(uint4)},
        {T.d_hdr, (T.n_steps + kRegsSpareSteps) * kRegsWaves * layout.head * (int64_t)sizeof(uint32_t)},
        {T.d_node, accumulators * (int64_t)sizeof(int32_t)},
        {T.d_row, accumulators * (int64_t)sizeof(int32_t)},
        {T.d_unit, T.n_units * (int64_t)sizeof(RegsUnit)},
        {T.d_part, T.n_parts * (int64_t)sizeof(RegsPart)},
        {T.d_sum, T.n_sums * (int64_t)sizeof(RegsSum)},
        {T.d_split, T.n_split * (int64_t)sizeof(RegsSplit)},
    };
    if (which < 0 || which >= (int32_t)std::size(tables)) return MAXK_INVALID_ARGUMENT;
    const auto [at, n] = tables[which];
    if (!out || n == 0) return n;
    if (bytes < n) return MAXK_INVALID_ARGUMENT;
    if (which == 0) std::memcpy(out, sizes, sizeof(sizes));
    else MAXK_HIP_TRY(hipMemcpy(out, at, (size_t)n, hipMemcpyDeviceToHost));
    return n;
}

MAXK_API int32_t maxk_graph_sweep_tables(const maxk_graph* g) { return g ? (int32_t)g->sweep_cache.size() : MAXK_INVALID_ARGUMENT; }

MAXK_API int64_t maxk_graph_limit_allocations(maxk_graph* g, int64_t bytes)
{
    if (!g) return MAXK_INVALID_ARGUMENT;
    g->test_alloc_limit = bytes;
    return g->test_denied;
}

int32_t maxk_last_hip_error(void) { return g_last_hip_error; }

MAXK_API int32_t maxk_version(void) { return 100; }

}  // extern "C"
