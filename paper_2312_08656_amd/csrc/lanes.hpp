// How a wavefront shares its lanes out over stored entries (forward and pull kernels).
#pragma once

#include <utility>

#include "common.hpp"

namespace maxk {
namespace {

// LANES lanes (8, 16, 32 or 64) work on an entry, a CBSR position each, in PASSES wave instructions; kWave / LANES entries are worked
// on side by side.  Lane groups whose last pass is not full repeat position k - 1: the same value to the same place.  The entries
// of a batch are held by the lanes themselves, a register of them in every 16 lanes (LANES = 8: in every quad), and an
// instruction takes entry E of its group by a data-parallel-primitive broadcast that is part of it.
template <int LANES_, int PASSES_>
struct FwdLanes {
    static constexpr int LANES = LANES_, PASSES = PASSES_, GROUPS = kWave / LANES;
    static constexpr int PER = LANES >= 16 ? 16 : 4;                   // entries of a group in one register
    static constexpr int BATCH = LANES >= 16 ? 16 : 8, HELD = BATCH / PER;  // entries of a group in a batch; registers that hold them
    static constexpr int STEP = LANES == 8 && PASSES == 1 ? 4 : PASSES >= 5 ? 1 : PASSES >= 3 ? 2 : 8 / PASSES;  // loaded together
    static constexpr int STEPS = BATCH / STEP, ROUNDS = STEP * PASSES;
    static_assert(STEPS % 2 == 0, "two sets of registers take turns");
    static constexpr bool WHOLE = LANES == kWave || PASSES == 1;       // the last pass is full
};

template <int I>
__device__ __forceinline__ uint32_t row16_lane(uint32_t x)  // lane I of the caller's 16 lanes
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x150 + I, 0xF, 0xF, true);
}

template <int PER, int I>
__device__ __forceinline__ uint32_t held_entry(uint32_t x)  // entry I of the register of the caller's 16 or 8 lanes or quad
{
    if constexpr (PER == 16) return row16_lane<I>(x);
    else if constexpr (PER == 4) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, I * 0x55, 0xF, 0xF, true);
    else return (uint32_t)__builtin_amdgcn_update_dpp((int)row16_lane<I>(x), (int)x, 0x158 + I, 0xF, 0xC, false);  // (upper eight: their own)
}

constexpr auto kAlways = [](auto) { return true; };

template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    [&]<int... I>(std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }(std::make_integer_sequence<int, N>{});
}

// Stored entries [begin, end) of a work item, a batch at a time: entry and weight of this lane's place in the batch at `base`.  Whole
// batches: a run of entries to each register of a group, so that the lanes of a load are next to each other; the last, shorter one: the
// groups take its entries in turn (the last entry again behind them).
template <class S>
struct EntryBatches {
    static constexpr int kBatch = S::GROUPS * S::BATCH;
    const int32_t* node;
    const float* weight;
    uint32_t end;
    uint32_t in_run, in_turn;

    __device__ __forceinline__ EntryBatches(const int32_t* n, const float* w, uint32_t e, int lane) : node(n), weight(w), end(e)
    {
        const int g = lane / S::LANES;
        in_run = (uint32_t)(g * S::PER + lane % S::PER);
        in_turn = (uint32_t)((lane % S::PER) * S::GROUPS + g);
    }
    __device__ __forceinline__ void fetch(uint32_t base, int2 (&e)[S::HELD]) const
    {
        const uint32_t from = batch_begin(base, end), most = end - 1u - from,
                       mine = most + 1u >= (uint32_t)kBatch ? in_run : in_turn;
#pragma unroll
        for (int r = 0; r < S::HELD; ++r) {
            const uint32_t p = min(mine + (uint32_t)(r * S::PER * S::GROUPS), most);
            e[r] = make_int2((node + from)[p], __float_as_int((weight + from)[p]));
        }
    }
};

// Runs `w` (hold, load<F, WIDE>, add<F>, settle) over the entries of a work item: the loads of the next STEP entries, of the next batch in
// the end, are under way while STEP entries are added.  wide: 64-bit offsets, nothing under way.
template <class S, class Wave>
__device__ __forceinline__ void run_item(Wave& w, const EntryBatches<S>& entries, int begin, int end, int g, bool wide)
{
    constexpr int kBatch = EntryBatches<S>::kBatch;
    if (begin >= end) return;
    uint32_t base = begin;
    int left = end - begin;
    int2 e[S::HELD];
    entries.fetch(base, e);
    typename Wave::Held cur = w.hold(e);
    typename Wave::Step s0, s1;
    if (wide) {
        while (left > 0) {
            static_for<S::STEPS>([&](auto i) {
                w.template load<decltype(i)::value * S::STEP, true>(cur, s0, [&](int n) { return n * S::GROUPS < left; });
                w.template add<decltype(i)::value * S::STEP>(cur, s0, [&](auto n) { return decltype(n)::value * S::GROUPS + g < left; });
            });
            base += kBatch;
            left -= kBatch;
            if (left > 0) {
                entries.fetch(base, e);
                cur = w.hold(e);
            }
        }
        return;
    }
    if (left >= kBatch) {
        entries.fetch(base + kBatch, e);
        w.template load<0>(cur, s0, kAlways);
        w.settle(s0);
        do {
            typename Wave::Held next;
            static_for<S::STEPS>([&](auto i) {
                constexpr int I = decltype(i)::value, F = I * S::STEP;
                typename Wave::Step& mine = I % 2 ? s1 : s0;
                typename Wave::Step& other = I % 2 ? s0 : s1;
                if constexpr (I + 1 < S::STEPS) {
                    w.template load<F + S::STEP>(cur, other, kAlways);
                } else {  // the first ones of the next batch (the last entry's again behind the last)
                    next = w.hold(e);
                    w.template load<0>(next, other, kAlways);
                    entries.fetch(base + 2 * kBatch, e);
                }
                w.template add<F>(cur, mine, kAlways);
            });
            cur = next;
            base += kBatch;
            left -= kBatch;
        } while (left >= kBatch);
    } else {
        w.template load<0>(cur, s0, [&](int n) { return n * S::GROUPS < left; });
    }
    if (left <= 0) return;
    static_for<S::STEPS>([&](auto i) {
        constexpr int I = decltype(i)::value, F = I * S::STEP;
        typename Wave::Step& mine = I % 2 ? s1 : s0;
        typename Wave::Step& other = I % 2 ? s0 : s1;
        if (F * S::GROUPS < left) {
            if constexpr (I + 1 < S::STEPS) w.template load<F + S::STEP>(cur, other, [&](int n) { return n * S::GROUPS < left; });
            w.template add<F>(cur, mine, [&](auto n) { return decltype(n)::value * S::GROUPS + g < left; });
        }
    });
}

}  // namespace
}  // namespace maxk
