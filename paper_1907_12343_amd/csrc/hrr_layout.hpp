// hrr_layout.hpp -- host-side choices of a traversal launch's layout (eye
// order key, work-queue layout, output chunk size, partial-chunk bound).
// Plain functions of the launch's sizes, unit-tested on the CPU.
#pragma once

#include <math.h>
#include <stdint.h>

#include "hrr_types.hpp"

namespace hrr {

// Eye-order key widths for n items holding `virtual_eyes` virtual eyes in all:
// Morton cells of about 2^11 or more virtual eyes each (at least two bits per
// axis where the bucket budget allows), then up to 9 bits of the shift class
// (no more than the tile values' significant bits), within kOrderMaxBuckets
// buckets.  bits = 0: no reordering.  On the 1920x1080 frame over 2^20 lights
// (3 bits per axis, 9 class bits) this runs 4-5 % faster than finer cells
// alone; a launch of 256 small items is insensitive to the split as long as
// cells have two or more bits per axis.
inline void order_key_bits(uint64_t n, uint64_t virtual_eyes, uint32_t tile_bits, uint32_t* bits_out,
                           uint32_t* rbits_out) {
    uint32_t bits = 0, rbits = 0;
    if (n > 0 && virtual_eyes > 0 && virtual_eyes < 0xFFFFFFFFull) {
        const uint64_t per_item = virtual_eyes / n > 0 ? virtual_eyes / n : 1;
        while (bits < 2 && (n << (3 * (bits + 1))) <= kOrderMaxBuckets) ++bits;
        while (bits && bits < 10 && (per_item >> (3 * (bits + 1))) >= (1u << 11) &&
               (n << (3 * (bits + 1))) <= kOrderMaxBuckets)
            ++bits;
        if (bits && tile_bits) {
            rbits = tile_bits < 9u ? tile_bits : 9u;
            while (rbits && (n << (3 * bits + rbits)) > kOrderMaxBuckets) --rbits;
        }
    }
    *bits_out = bits;
    *rbits_out = rbits;
}

// Whether a launch orders its eyes at all: the ordering pass (five small
// kernels and their set-up) costs about 35 us per call, which only pays when
// the launch has enough work for cache locality to matter.  `cost` is the
// launch's estimated work, the sum over items of virtual eyes x
// n_lights^0.6 (the cost model of the work queues).  4096 eyes x 1024 lights
// (cost 2.6e5): 0.134 ms per call unordered against 0.170 ordered; 4096 of the
// frame's eyes x 2^20 lights (cost 1.7e7): 1.37 unordered against 1.34
// ordered, and ordering halves the time from 2^15 such eyes on.
constexpr double kOrderMinCost = 2097152.0;   // 2^21
inline bool order_pays(double cost) { return cost >= kOrderMinCost; }

// Work-queue layout: launches of several items with 2^19 or more tasks use
// interleaved chunks of 2^13 tasks (queue q owns chunks q, q + 8, ...), so all
// XCDs work on the same heavy items at a time and the Infinity Cache holds
// fewer hierarchies at once (256 caches: kernel 70.3 -> 66.5 ms); others use
// eight contiguous slices of equal cost.  Returns the chunk shift, 0 for
// slices.  (The block walk always takes slices: its waves pass through items
// faster, and with slices only one XCD's waves pass through most items, each
// leaving two or three atomics on the item's counters.  64 caches: 4.8 ms with
// slices against 8.7 with chunks of 2^8 tasks.)
inline uint32_t queue_interleave_shift(uint64_t n, uint64_t tasks) {
    return (n > 1 && tasks >= (1ull << 19)) ? 13u : 0u;
}

// Whether the block walk takes an item of the default method: its reciprocal
// bound needs s within the range of the product-form test (s / d^2 a normal
// number); an s outside it runs the node walk, whose tests fall back to the
// IEEE division.
inline bool block_walk_takes(float s) { return s >= 0x1p-60f && s <= 0x1p60f; }
// Estimated work of one eye against n_lights lights, in arbitrary units (the
// growth of the walk's steps).
inline double eye_cost(uint32_t n_lights) { return pow((double)(n_lights > 1u ? n_lights : 1u), 0.6); }

// log2 of the eyes per task of an item in a block-walk launch of total work
// `launch_cost` (the sum over items of virtual eyes x eye_cost): tasks of
// equal work, about kTasksPerWave of them per resident wave (eyes differ in
// work by far more than the estimate says, and a launch ends with its longest
// last task), but at least kMinTaskCost each (a task costs an atomic and an
// eye upload, and a wave that leaves an item two or three more) and at most
// 64 eyes, a wave's eye slots.  A launch of less than kFewTasks times
// kMinTaskCost still makes about kFewTasks tasks, or one per eye: it would else
// leave the GPU to a few waves (us a call into a buffer of 2^26 pairs, tasks of
// kMinTaskCost / kFewTasks of them / the node walk: 300 eyes x 2^18 lights at s
// = 1e-2 1724 / 326 / 1611, at s = 1e-8 60 / 75 / 112; 3000 eyes x 2^14 lights
// at s = 1e-4 146 / 130 / 169).  More of them cost more in the compaction of
// their partly filled chunks than they gain (one task per resident wave: 307 us
// for 30,000 eyes x 2^10 lights, 101 as it is).
//
// A launch with dense output is small: it aims at kDenseTasks tasks, one per
// wave, and where whole eyes make fewer than a quarter of that, an eye's walk is
// cut into the 4 or 16 blocks of the tree's first levels.
constexpr double kTasksPerWave = 32.0;
constexpr double kMinTaskCost = 16384.0;
constexpr double kFewTasks = 512.0;
constexpr double kDenseTasks = 4096.0;
inline void block_task_split(uint32_t n_lights, double launch_cost, uint64_t resident_waves, bool dense,
                             uint32_t* task_shift, uint32_t* sub_log) {
    const double want = dense ? fmin(launch_cost / kDenseTasks, kMinTaskCost)
                              : fmax(launch_cost / (kTasksPerWave * (double)resident_waves),
                                     fmin(launch_cost / kFewTasks, kMinTaskCost));
    const double target = want / eye_cost(n_lights);   // eyes per task
    uint32_t shift = 0, sub = 0;
    if (dense) {
        while (shift < 6u && (double)(1u << shift) < target) ++shift;
        const uint32_t log = block_tree_log(n_lights);
        while (sub < 4u && target * (double)(4u << sub) <= 1.0 && log - block_leaf_log(log) >= sub + 6u) sub += 2;
    } else {
        while (shift < 6u && (double)(2u << shift) <= target) ++shift;
    }
    *task_shift = shift;
    *sub_log = sub;
}
// Whether a block-walk launch writes its output dense, one atomic per 512
// pairs or wave (see cull_kernel).  us a call, dense / chunks and compaction:
// 5001 eyes x 2^20 lights, 1.4e5 pairs 83 / 201; 9.4e6 pairs 300 / 413; 1.8e7
// pairs 892 / 988; 3.8e7 pairs 1087 / 869, bound by the atomics.  Counting
// calls take it for its set-up, up to the size where resident waves count more
// (its LDS leaves 5 blocks to a CU against 8).
inline bool block_walk_dense(uint64_t capacity, double launch_cost) {
    return capacity ? capacity <= (1ull << 24) : launch_cost < 268435456.0;
}
// The pairs that an item can store: no more than its eyes have lights, however
// large its buffer.  A small launch into a large buffer is dense by this (300
// eyes x 2^12 lights into 2^25 pairs: 118 us in chunks, 37 dense).
inline uint64_t item_room(uint64_t capacity, uint64_t virtual_eyes, uint32_t n_lights) {
    const uint64_t all = virtual_eyes * n_lights;   // below 2^32 * 2^25
    return capacity < all ? capacity : all;
}

// Estimated work of a launch (the sum over its items of virtual eyes x
// eye_cost), its virtual eyes and the pairs that it can store.
struct LaunchSize {
    double cost = 0.0;
    uint64_t eyes = 0, room = 0;
    void add(uint64_t virtual_eyes, uint32_t n_lights, uint64_t capacity) {
        const uint64_t r = item_room(capacity, virtual_eyes, n_lights);
        cost += (double)virtual_eyes * eye_cost(n_lights);
        eyes = virtual_eyes > ~0ull - eyes ? ~0ull : eyes + virtual_eyes;
        room = r > ~0ull - room ? ~0ull : room + r;
    }
};

// Whether lights of this spread (hrr_types.hpp) are too scattered for the block
// walk: an eye inside a smallest block's box must test all its lights, where the
// node walk still has the boxes of fewer lights below it.  Speed of the block
// walk relative to the node walk, scenes 1, 5, 10 and 100 times as large as the
// box that orders their lights, and beside it:
//   dense output: spread 1 .. 4 at least 2; 3,000 eyes 2.2 .. 5.5 at spread 2^8,
//     0.94 .. 1.5 at 2^13 (2^18 lights), 0.71 at 2^15 (2^20); 30,000 eyes 1.03 ..
//     2.5 at 2^8, 0.98 .. 1.4 at 2^9, 0.43 .. 1.3 from 2^10; below 2^16 lights
//     and in small launches hardly under 1, as blocks that are cut among several
//     waves make up for it (5 items of 300 eyes, spread 2^15, 2^20 lights: 0.67);
//   chunks: 3,000 .. 30,000 eyes 0.9 .. 1.8 at 2^6 and 2^7, 0.6 .. 1.8 at 2^8,
//     0.17 .. 0.9 from 2^10, and 0.5 with 2^12 lights where an eye is in every
//     second block; 300,000 eyes 0.9 .. 1.8 up to 2^10, 0.6 .. 0.9 from 2^11;
//     below 2^12 lights at least 1.
inline bool node_walk_scattered(float spread, uint32_t n_lights, const LaunchSize& size, bool dense) {
    if (dense) {
        const double met = (double)spread * (double)size.eyes;   // blocks that the launch's eyes stand in
        return n_lights >= (1u << 16) && spread >= 512.0f && (met >= 6e7 || (met >= 2.4e7 && size.cost >= 1e7));
    }
    const uint32_t n_blocks = block_tree_lights(n_lights) >> block_leaf_log(block_tree_log(n_lights));
    const float bound = size.eyes < (1u << 17) ? fminf(256.0f, (float)n_blocks / 8.0f) : 2048.0f;
    return n_lights >= (1u << 12) && spread >= bound;
}

// How often one wave can leave one item (publishing a partly filled chunk).
// A wave visits each queue once (cyclic order from its own) and takes a
// queue's tasks in increasing order, so within one queue visit the items it
// meets are nondecreasing and it leaves an item at most once.  Contiguous
// slices are in task order too: at most twice per item (the one wrap), once
// in a one-item launch; interleaved chunks: at most once per queue visit.
inline uint64_t departures_per_wave(uint64_t n, uint32_t interleave_shift) {
    return interleave_shift ? kQueues : (n > 1 ? 2 : 1);
}

// Eyes per wavefront for a hierarchy of n_lights lights when neither the
// caller nor the tuner fixes it.  Small hierarchies give an eye only tens to
// hundreds of node visits, too few to keep 64 lanes busy (one eye per wave:
// 13 % of the lanes active at 2^10..2^12 lights, 37 % at 2^14..2^16, 89 % at
// 2^18..2^20), so several eyes share a wave.  Thresholds measured on batched
// launches of mixture caches at s = 1e-4 (kernel ms at 1 / 4 / 8 eyes per wave:
// 2^10..2^12 lights 3.82 / 1.40 / 0.76, 2^14..2^16 6.34 / 3.37 / 3.11,
// 2^16..2^17 3.36 / 3.04 / 3.08, 2^17..2^18 8.90 / 8.94 / 9.08, 2^18..2^20
// 40.4 / 45.2 / 51.3).
inline uint32_t default_eyes_per_wave(uint32_t n_lights) {
    return n_lights >= (1u << 17) ? 1u : n_lights >= (1u << 16) ? 4u : 8u;
}

// LDS stack entries per wave when neither the caller nor the tuner fixes
// them.  One eye per wave also keeps a 4160-byte record area in LDS; 192
// entries (1.5 KB) leave room for 7 waves per SIMD in 160 KB, 256 entries
// for 6 (frame, power-of-two splits: 123.7 ms at 192 entries against 127.9 ms
// at 256 and 154.3 ms at 512).  Several eyes per wave run at 96 registers (5
// waves per SIMD) with their eyes in LDS, where 512 entries cost nothing.
inline uint32_t default_stack_entries(uint32_t eyes_per_wave) {
    return eyes_per_wave == 1 ? 192u : 512u;
}

// Stack sizes the autotuner tries for a shape, in order of preference.
inline void tune_stack_candidates(uint32_t eyes_per_wave, uint32_t out[3]) {
    if (eyes_per_wave == 1) {
        out[0] = 192; out[1] = 256; out[2] = 512;
    } else {
        out[0] = 512; out[1] = 256; out[2] = 1024;
    }
}

// Whether a block-walk launch orders its eyes: `cost` is the work of its items
// whose light blocks outgrow an XCD's 4 MB L2 (2^18 lights and more).  ms a
// call, ordered / in index order: 2^16 eyes x 2^20 lights at s = 1e-6 (cost
// 2^28) 0.21 / 0.19, 2^18 eyes 0.51 / 0.57, at s = 1e-4 3.6 / 9.1; 2^20 eyes x
// 2^18 lights at s = 1e-4 4.3 / 4.8; with 2^16 lights and fewer the ordering
// pass is never won back (2^20 eyes x 2^16 lights 2.46 / 2.33).
inline bool block_order_pays(double cost) { return cost >= 268435456.0; }
inline bool block_order_counts(uint32_t n_lights) { return n_lights >= (1u << 18); }

// Output chunk size of an item: about sixteen chunks per wave that touches
// the item, 2^kMinChunkShift .. 2^kMaxChunkShift pairs.
inline uint32_t chunk_shift_for(uint64_t capacity, uint64_t touching_waves) {
    uint32_t shift = kMinChunkShift;
    while (shift < kMaxChunkShift && (capacity >> (shift + 1)) >= 16 * touching_waves) ++shift;
    return shift;
}
// The same for the block walk: about four chunks per wave.  Its launches end
// sooner, so the chunk atomics of one address, 13 ns each, weigh more than the
// compaction of larger tails (2^18 eyes x 2^16 lights, 3.8e7 pairs: 2.01 ms at
// sixteen, 0.87 at four; 1.5e8 pairs 2.2 and 1.74; the frame does not change).
inline uint32_t block_chunk_shift(uint64_t capacity, uint64_t touching_waves) {
    uint32_t shift = kMinChunkShift;
    while (shift < kMaxChunkShift && (capacity >> (shift + 1)) >= 4 * touching_waves) ++shift;
    return shift;
}

}  // namespace hrr
