// hrr_kernels.hip -- gfx950 kernels for hierarchical Russian roulette with a
// rotated base-2 radical inverse (Pantaleoni, "Blue-Noise Dithered QMC
// Hierarchical Russian Roulette").
//
//   rmq_kernel       range-minimum queries (Section 1, v(a,b); Section 2,
//                    Algorithms 2-3), eight per thread, streaming u32 arrays.
//   cull_kernel      the default traversal: persistent wavefronts that bound
//                    aligned blocks of lights and list their candidates in
//                    closed form (see "block walk").
//   traverse_kernel  the node walk (statistics, the other range-minimum
//                    methods, extreme s): persistent wavefronts that pull (item, eye group) tasks
//                    from eight per-XCD work queues and cull every eye's pairs
//                    by a top-down walk of its item's light hierarchy
//                    (Section 1).
//   around it        the eye order (bucket keys, a multi-block scan, scatter)
//                    and the compaction that makes every item's output dense
//                    after a traversal (compact_plan_kernel,
//                    compact_move_kernel).
//
// Wavefront design of the node walk.  One wave owns a group of 1..8 eyes.  Its stack of
// pending hierarchy nodes lives in LDS and is shared by the 64 lanes: each
// iteration pops up to 64 nodes (one per lane), each lane obtains its node's
// 64-byte record (both children's boxes; neighbouring lanes fetch their two
// records as shared 32-byte halves), derives the children's range minima
// -- the child that contains the parent's argmin inherits it, the other needs
// one range-minimum query -- bounds both children, and the survivors are
// pushed back with ballot/mbcnt compaction.  Leaves with one light are tested
// exactly at the parent; accepted pairs go straight from the lanes into an
// output chunk the wave owns (one atomic per chunk of thousands of pairs, see
// emit2).  The stack spills in halves to a per-wave region
// of device memory when it would overflow LDS; its size is bounded by
// 128 entries per tree level (see stack_spill).
//
// Floating point: every acceptance probability is computed in binary32 with
// separately rounded operations (no contraction) and an IEEE division, so that
// a one-light leaf's test is bit-identical to the all-pairs definition.
#include <hip/hip_runtime.h>

#include <mutex>

#include "hrr_compact.hpp"
#include "hrr_devbuild.hpp"
#include "hrr_rmq.hpp"
#include "hrr_scan.hpp"
#include "hrr_types.hpp"

#pragma clang fp contract(off)

namespace hrr {

// ---------------------------------------------------------------------------
// wavefront helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// lanes (of the active ones) whose p holds; the builtin takes the condition as
// a lane mask directly (the int-valued __ballot materialises it in a register
// and compares it again)
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// number of set bits of m in lanes below this one
__device__ __forceinline__ uint32_t count_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ float unif(float x) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// Order LDS traffic of one wave across lanes: the wave executes in lock step
// and LDS serves one wave's requests in order, so only compiler reordering
// has to be prevented.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// acceptance bound
// ---------------------------------------------------------------------------

// squared distance from the eye to the box [lo, hi] (0 inside), summed
// (x + y) + z; for a one-point box this is the pair's own d^2 bit for bit.
// Hierarchy records and lights always live in device global memory; loading
// them through an address-space-1 pointer makes the compiler emit global
// loads instead of generic (flat) ones, which would also tie up the LDS
// counter that the stack operations wait on.
typedef float f32x4 __attribute__((ext_vector_type(4)));
// DPP control: quad_perm(1, 0, 3, 2) -- every lane reads its pair partner.
constexpr int kDppSwapPairs = 0xB1;

__device__ __forceinline__ float swap_pairs(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kDppSwapPairs, 0xF, 0xF, false));
}
__device__ __forceinline__ float4 swap_pairs(float4 v) {
    return make_float4(swap_pairs(v.x), swap_pairs(v.y), swap_pairs(v.z), swap_pairs(v.w));
}

__device__ __forceinline__ float4 load_global4(const float4* p, uint32_t i) {
    const f32x4 v = ((const __attribute__((address_space(1))) f32x4*)(p))[i];
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ float box_d2(float ex, float ey, float ez, float lx, float ly, float lz,
                                        float hx, float hy, float hz) {
    const float dx = fmaxf(fmaxf(lx - ex, ex - hx), 0.0f);
    const float dy = fmaxf(fmaxf(ly - ey, ey - hy), 0.0f);
    const float dz = fmaxf(fmaxf(lz - ez, ez - hz), 0.0f);
    const float x2 = dx * dx;
    const float y2 = dy * dy;
    const float z2 = dz * dz;
    return (x2 + y2) + z2;
}

// p = min(1, (s / d2) * mult).  mult = 1 for an exact one-light test; for a
// multi-light box mult = 1 + 2^-20, a safety factor on the bound (every step
// above is monotone, so the box bound is already >= each light's p).
__device__ __forceinline__ float accept_p(float s, float d2, float mult) {
    float q = s / d2;
    q = q * mult;
    return fminf(q, 1.0f);
}

// Russian roulette with a 32-bit fixed-point random number: keep iff
// v / 2^32 < p, i.e. v < ceil(p * 2^32) (exact: the scaling is a power of 2).
__device__ __forceinline__ bool keeps(uint32_t v, float p) {
    if (p >= 1.0f) return true;
    return v < (uint32_t)ceilf(p * 4294967296.0f);
}

constexpr float kBoxMargin = 1.0f + 0x1p-20f;

// ---- product-form keep test ------------------------------------------------
//
// With x = fl(s / d2) 2^32 the pair is kept iff v < x (v is an integer, so
// v < ceil(x) is the same as v < x).  Instead of the IEEE quotient (about ten
// VALU instructions) the kernel compares the product P = fl(fl(v) d2) with
// two per-item constants, t_cull >= S (1 + 2^-18) and t_keep <= S (1 - 2^-18),
// S = s 2^32.  Each of fl(v), the product and fl(s / d2) has a relative error
// of at most 2^-24, so
//   P > t_cull  implies  v > (s / d2) 2^32 (1 + 2^-24) >= x   (culled), and
//   P < t_keep  implies  v < (s / d2) 2^32 (1 - 2^-24) <= x   (kept).
// For d2 <= s (p = 1) the first never holds, since fl(v) d2 <= 2^32 s.
// A box at squared distance d2 bounds every light inside it (each light's
// squared distance, computed with the same monotone binary32 steps, is at
// least d2), so "P > t_cull" culls a whole subtree safely; anything else
// keeps the box.  A one-light test whose product falls between the two
// constants (a relative band of about 2^-17 around the threshold) decides
// with the IEEE quotient.  The product form is used only for
// d2 <= d2_fast = s 2^60 (s / d2 stays a normal number, P cannot overflow);
// beyond it, and for s outside [2^-60, 2^60], the IEEE path decides.

// Product-form part of the keep test, with selects only: sets `keep` and
// returns false when decided, returns true when the IEEE path must decide.
__device__ __forceinline__ bool rr_fast(uint32_t v, const ItemDesc& D, float d2, bool exact, bool& keep) {
    const float P = (float)v * d2;
    const bool fast = d2 <= D.d2_fast;
    const bool cull = fast && P > D.t_cull;
    const bool sure = fast && (!exact || P < D.t_keep);
    keep = !cull;
    return !cull && !sure;
}

// Keep test of value v at squared distance d2.
//   exact = true : one light; the result equals keeps(v, min(1, s / d2)).
//   exact = false: a box; false only if no light in the box can keep v.
__device__ __forceinline__ bool rr_test(uint32_t v, const ItemDesc& D, float d2, bool exact) {
    if (d2 <= D.d2_fast) {
        const float P = (float)v * d2;
        if (P > D.t_cull) return false;
        if (!exact || P < D.t_keep) return true;
    }
    return keeps(v, accept_p(D.s, d2, exact ? 1.0f : kBoxMargin));
}

// Fixed-point golden-ratio lattice alpha = round(2^32 (sqrt(5) - 1) / 2).
constexpr uint32_t kGoldenAlpha = 2654435769u;

// ---------------------------------------------------------------------------
// range-minimum kernel
// ---------------------------------------------------------------------------

template <int METHOD>
__device__ __forceinline__ void rmq_one(uint32_t a, uint32_t b, uint32_t R, uint32_t& k, uint32_t& v,
                                        uint32_t& bad) {
    if (a < b) {
        k = rmq<METHOD>(a, b, threshold_index(R));
        v = rotated(k, R);
    } else {
        k = b;
        v = 0xFFFFFFFFu;
        ++bad;
    }
}

// Four queries per lane per step through 16-byte loads when every array is
// 16-byte aligned (vec != 0); the scalar tail and unaligned arrays go one
// query at a time.  Every array is touched once, so loads and stores are
// non-temporal (2^28 queries: 0.895 ms against 0.970 ms with ordinary ones;
// non-temporal stores alone 0.96 ms, loads alone 0.98 ms).
constexpr uint32_t kRmqGroups = 1;   // 4-query groups per thread (2^28 queries: 1: 0.925 ms, 2: 0.941, 4: 0.955)

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 load_stream4(const uint4* p, uint64_t i) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p) + i);
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void store_stream4(uint4* p, uint64_t i, uint4 x) {
    const u32x4 v = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p) + i);
}

template <int METHOD>
__global__ __launch_bounds__(256) void rmq_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B,
                                                  const uint32_t* __restrict__ R, uint64_t n,
                                                  uint32_t* __restrict__ K, uint32_t* __restrict__ V,
                                                  unsigned long long* __restrict__ n_bad, int vec) {
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint32_t bad = 0;
    uint64_t done = 0;
    if (vec) {
        const uint64_t n4 = n >> 2;
        const uint4* A4 = reinterpret_cast<const uint4*>(A);
        const uint4* B4 = reinterpret_cast<const uint4*>(B);
        const uint4* R4 = reinterpret_cast<const uint4*>(R);
        uint4* K4 = reinterpret_cast<uint4*>(K);
        uint4* V4 = reinterpret_cast<uint4*>(V);
        // kRmqGroups 4-query groups per thread, all loads first; block b
        // covers groups [b, b + 1) x blockDim x kRmqGroups, so every load and
        // store instruction of a block is contiguous
        for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x * kRmqGroups; base < n4;
             base += stride * kRmqGroups) {
            uint4 a[kRmqGroups], b[kRmqGroups], r[kRmqGroups];
#pragma unroll
            for (uint32_t g = 0; g < kRmqGroups; ++g) {
                const uint64_t q = base + g * blockDim.x + threadIdx.x;
                if (q < n4) {
                    a[g] = load_stream4(A4, q);
                    b[g] = load_stream4(B4, q);
                    r[g] = load_stream4(R4, q);
                }
            }
#pragma unroll
            for (uint32_t g = 0; g < kRmqGroups; ++g) {
                const uint64_t q = base + g * blockDim.x + threadIdx.x;
                if (q < n4) {
                    uint4 k, v;
                    rmq_one<METHOD>(a[g].x, b[g].x, r[g].x, k.x, v.x, bad);
                    rmq_one<METHOD>(a[g].y, b[g].y, r[g].y, k.y, v.y, bad);
                    rmq_one<METHOD>(a[g].z, b[g].z, r[g].z, k.z, v.z, bad);
                    rmq_one<METHOD>(a[g].w, b[g].w, r[g].w, k.w, v.w, bad);
                    store_stream4(K4, q, k);
                    store_stream4(V4, q, v);
                }
            }
        }
        done = n4 << 2;
    }
    for (uint64_t q = done + tid; q < n; q += stride) {
        uint32_t k, v;
        rmq_one<METHOD>(__builtin_nontemporal_load(A + q), __builtin_nontemporal_load(B + q),
                        __builtin_nontemporal_load(R + q), k, v, bad);
        __builtin_nontemporal_store(k, K + q);
        __builtin_nontemporal_store(v, V + q);
    }
    if (n_bad) {
        const uint64_t m = ballot(bad != 0);
        if (m) {
            // wave-reduce the few non-zero counts
            uint32_t tot = bad;
            for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o);
            if (lane_id() == 0) atomicAdd(n_bad, (unsigned long long)tot);
        }
    }
}


// ---------------------------------------------------------------------------
// traversal kernel
// ---------------------------------------------------------------------------

struct EyeState {
    float ex, ey, ez;
    uint32_t R;     // rotation r_j (+ extras), fixed point
    uint32_t kr;    // threshold index Phi_2^{-1}(1 - r_j)
    uint32_t u;     // virtual eye index emitted as the pair's first component
};

// Record fetch of the walk.  One eye per wave: the four lanes of a quad
// fetch their four 64-byte records as 16-byte quarters, so every load of a
// quad touches a single record, and the quarters go straight from memory into
// LDS (global_load_lds_dwordx4 writes lane L's 16 bytes at the instruction's
// LDS base + 16 L), where each lane reads its own record back.  The area holds
// one 1040-byte slab per record slot t of a quad: 1024 bytes for the 64 lanes
// and 16 bytes that stagger the slabs over the LDS banks.  Several eyes per
// wave (which keep their eyes in LDS and run at lower occupancy): lanes 2i,
// 2i + 1 fetch both of their records as 32-byte halves and swap halves with a
// DPP lane exchange.
constexpr uint32_t kSlab = 1040;
constexpr uint32_t kXposeBytes = 4 * kSlab;
template <int EPW>
struct FetchOf {
    static constexpr bool quad_lds = EPW == 1;
};

constexpr uint32_t kEyeTableBytes = 8 * 8 * sizeof(uint32_t);   // 8 words per eye slot

// LDS of one wave: the stack ring, then the eye table (several eyes per wave)
// or the record area (one eye per wave).
struct WaveLds {
    uint2* stack;
    uint32_t* eyes;   // 8 words per slot
    unsigned char* xpose;
};

// ---- per-wave stack in LDS with spill to device memory ----
//
// Logical positions [0, g) live in the wave's spill region, [g, g + n) in an
// LDS ring of cap entries (cap a multiple of 64, at least 192); the entry at
// logical position g sits in ring slot `base`, the next ones follow it round
// the ring.  Stack memory moves in units of 64 entries, one per lane, so a
// lane always re-reads exactly what it wrote.  One unit is always enough:
// after a pop the ring holds at most cap - 64 entries (or none), a step pushes
// at most 128, so an overflowing push needs at most 64 more slots, and it
// only overflows when the ring holds more than cap - 128 >= 64 entries.
//
// Size bound.  Pops take the top <= 64 entries (lanes in stack order) and
// each pushes its surviving children next to each other, so depths never
// decrease from bottom to top.  A pop that reaches an entry of depth d - 1
// also removes every entry of depth >= d above it; hence all entries of depth
// d come from one pop and number at most 128, and the stack never holds more
// than 128 * (max depth + 1) entries.
constexpr uint32_t kStackUnit = 64;

struct StackState {
    uint32_t g;      // entries in device memory
    uint32_t n;      // entries in LDS
    uint32_t base;   // ring slot of logical position g
    uint32_t max_total;
    uint32_t spills;
};

// ring slot of x in [0, 2 cap): x or x - cap
__device__ __forceinline__ uint32_t ring(uint32_t x, uint32_t cap) { return min(x, x - cap); }

__device__ __forceinline__ bool stack_spill(StackState& st, const WaveLds& L, uint2* spill, uint32_t cap,
                                            uint32_t spill_cap, uint32_t* err) {
    if (st.g + kStackUnit > spill_cap) {
        if (lane_id() == 0) atomicOr(err, (uint32_t)ERR_SPILL_OVERFLOW);
        return false;
    }
    wave_sync();
    spill[st.g + lane_id()] = L.stack[ring(st.base + lane_id(), cap)];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    st.g += kStackUnit;
    st.n -= kStackUnit;
    st.base = ring(st.base + kStackUnit, cap);
    ++st.spills;
    return true;
}

__device__ __forceinline__ void stack_refill(StackState& st, const WaveLds& L, const uint2* spill, uint32_t cap) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    st.g -= kStackUnit;
    st.base = ring(st.base + cap - kStackUnit, cap);
    L.stack[ring(st.base + lane_id(), cap)] = spill[st.g + lane_id()];
    wave_sync();
    st.n += kStackUnit;
    ++st.spills;
}

// ---- pair output in per-wave chunks ----
//
// An item's output positions are cut into chunks of 2^chunk_shift pairs.  A
// wave takes a whole chunk from the item's chunk counter (one device-scope
// atomic per chunk instead of one per flush: a single address serialises
// those atomics) and writes its accepted pairs into it directly from the
// lanes, compacted with ballot/mbcnt.  A wave leaving an item publishes its
// partly filled chunk as (chunk, fill) (the launch bounds how often a wave can
// leave an item), so that the compaction kernels can move the pairs found
// past the final count into those holes.  Positions at or
// past the caller's capacity go to a library slack area, positions past that
// are dropped (the count stays exact).
constexpr unsigned long long kNoChunk = ~0ull;

struct OutState {
    unsigned long long chunk;   // current chunk, or kNoChunk
    unsigned long long count;   // pairs emitted for the current item
    uint2* wp;                  // first pair slot of the chunk when it lies wholly in one buffer
    float* ww;                  // same for the weights
    uint32_t fill;
};

__device__ __forceinline__ unsigned long long uni64(unsigned long long x) {
    return ((unsigned long long)uni((uint32_t)(x >> 32)) << 32) | uni((uint32_t)x);
}

__device__ __forceinline__ unsigned long long alloc_chunk(const ItemDesc& D) {
    unsigned long long c = 0;
    if (lane_id() == 0) c = atomicAdd(D.counters + CNT_CHUNKS, 1ull);
    return uni64(c);
}

// Pairs and weights are written once and not read again by the launch:
// non-temporal stores keep them from displacing node records in the caches
// (frame 144.5 -> 141.9 ms, 256-cache batch 57.2 -> 55.8 ms).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Stores go through global (address-space 1) pointers: a generic pointer
// makes them flat stores, which also count against the LDS counter that every
// stack access of the walk waits on.
typedef __attribute__((address_space(1))) u32x2 g_u32x2;
typedef __attribute__((address_space(1))) float g_f32;

__device__ __forceinline__ void put_pair(uint2* p, unsigned long long i, uint2 x) {
    const u32x2 v = {x.x, x.y};
    __builtin_nontemporal_store(v, (g_u32x2*)(p) + i);
}

__device__ __forceinline__ void put_weight(float* p, unsigned long long i, float w) {
    __builtin_nontemporal_store(w, (g_f32*)(p) + i);
}

// Make `c` the current chunk; direct pointers when the whole chunk lies below
// the capacity or inside the slack area (a chunk that straddles the capacity
// or the end of the slack takes the per-pair path).
template <bool W>
__device__ __forceinline__ void set_chunk(OutState& O, const ItemDesc& D, unsigned long long c) {
    O.chunk = c;
    O.wp = nullptr;
    O.ww = nullptr;
    if (c == kNoChunk) return;
    const unsigned long long p0 = c << D.chunk_shift;
    const unsigned long long C = 1ull << D.chunk_shift;
    if (p0 + C <= D.capacity) {
        O.wp = reinterpret_cast<uint2*>(D.pairs) + p0;
        if (W) O.ww = D.weights + p0;
    } else if (p0 >= D.capacity && p0 - D.capacity + C <= D.slack) {
        O.wp = reinterpret_cast<uint2*>(D.slack_pairs) + (p0 - D.capacity);
        if (W) O.ww = D.slack_weights + (p0 - D.capacity);
    }
}

template <bool W>
__device__ __forceinline__ void store_pair(const ItemDesc& D, unsigned long long p, uint2 pr, float w) {
    if (p < D.capacity) {
        put_pair(reinterpret_cast<uint2*>(D.pairs), p, pr);
        if (W) put_weight(D.weights, p, w);
    } else if (p - D.capacity < D.slack) {
        const unsigned long long q = p - D.capacity;
        put_pair(reinterpret_cast<uint2*>(D.slack_pairs), q, pr);
        if (W) put_weight(D.slack_weights, q, w);
    }
}

// Emit up to two pairs per lane, compacted over the wave (uniform control
// flow): every lane's first pair, then every lane's second, so that each of the
// two store instructions writes one contiguous run.  (With a lane's two pairs
// side by side, both instructions wrote every cache line in part: 1.52 bytes
// reached memory per byte of pairs.)  A step holds at most 128 pairs and a
// chunk at least 128, so a step crosses at most one chunk boundary.
template <bool W>
__device__ __forceinline__ void emit2(OutState& O, const ItemDesc& D, bool e0, uint2 p0, float w0, bool e1, uint2 p1,
                                      float w1) {
    const uint64_t m0 = ballot(e0), m1 = ballot(e1);
    const uint32_t cnt = (uint32_t)(__popcll(m0) + __popcll(m1));
    if (cnt == 0) return;
    if (D.capacity == 0) {   // counting launch: nothing is stored
        O.count += cnt;
        return;
    }
    if (O.chunk == kNoChunk) {
        set_chunk<W>(O, D, alloc_chunk(D));
        O.fill = 0;
    }
    const uint32_t shift = D.chunk_shift;
    const uint32_t C = 1u << shift;
    const uint32_t pos0 = O.fill + count_below(m0);
    const uint32_t pos1 = O.fill + (uint32_t)__popcll(m0) + count_below(m1);
    if (O.wp && uni(O.fill) + cnt <= C) {
        if (e0) {
            put_pair(O.wp, pos0, p0);
            if (W) put_weight(O.ww, pos0, w0);
        }
        if (e1) {
            put_pair(O.wp, pos1, p1);
            if (W) put_weight(O.ww, pos1, w1);
        }
        O.fill += cnt;
        O.count += cnt;
        if (O.fill == C) set_chunk<W>(O, D, kNoChunk);
        return;
    }
    unsigned long long next = kNoChunk;
    if (O.fill + cnt > C) next = alloc_chunk(D);
    const unsigned long long base = O.chunk << shift;
    const unsigned long long nbase = next << shift;
    if (e0) store_pair<W>(D, pos0 < C ? base + pos0 : nbase + (pos0 - C), p0, w0);
    if (e1) store_pair<W>(D, pos1 < C ? base + pos1 : nbase + (pos1 - C), p1, w1);
    O.count += cnt;
    O.fill += cnt;
    if (O.fill >= C) {
        O.fill -= C;
        set_chunk<W>(O, D, next);
    }
}

// A wave leaves an item: publish its count and its partly filled chunk.
__device__ __forceinline__ void close_item(OutState& O, const ItemDesc& D, uint32_t* err) {
    if (lane_id() == 0) {
        if (O.chunk != kNoChunk && O.fill > 0) {
            const unsigned long long at = atomicAdd(D.counters + CNT_PARTIALS, 1ull);
            if (at < D.partial_cap) {
                D.partials[2 * at] = O.chunk;
                D.partials[2 * at + 1] = O.fill;
            } else {
                atomicOr(err, (uint32_t)ERR_PARTIALS_OVERFLOW);
            }
        }
        if (O.count) atomicAdd(D.counters + CNT_PAIRS, O.count);
    }
    O.chunk = kNoChunk;
    O.wp = nullptr;
    O.ww = nullptr;
    O.fill = 0;
    O.count = 0;
}

__device__ __forceinline__ EyeState load_eye(const ItemDesc& D, const uint32_t* tile, uint32_t u) {
    EyeState E;
    const uint32_t ns = D.n_samples;
    const uint32_t j = ns > 1 ? u / ns : u;
    const uint32_t n = ns > 1 ? u - j * ns : 0u;
    E.ex = D.eyes[3u * j + 0];
    E.ey = D.eyes[3u * j + 1];
    E.ez = D.eyes[3u * j + 2];
    const uint32_t pix = D.pixel_base + j;
    const uint32_t x = pix % D.width;
    const uint32_t y = pix / D.width;
    uint32_t R = tile[(x & 63u) * 64u + (y & 63u)] + D.shift_offset;
    if (ns > 1) R += D.psi_s0 + n * kGoldenAlpha;
    E.R = R;
    E.kr = threshold_index(R);
    E.u = u;
    return E;
}

// Exact per-light tests of the leaf children that survived their box bound
// and hold more than one light.  Lane-local loops; emissions are compacted
// every step.
template <bool W>
__device__ __forceinline__ void leaf_lights(OutState& O, const ItemDesc& D, const EyeState& E, uint32_t la,
                                            uint32_t ln, uint32_t ra, uint32_t rn, uint64_t& tests) {
    const uint32_t total = ln + rn;
    for (uint32_t q = 0; ballot(q < total); ++q) {
        const bool act = q < total;
        bool emit = false;
        uint32_t i = 0;
        float w = 0.0f;
        if (act) {
            i = q < ln ? la + q : ra + (q - ln);
            const float4 P = load_global4(reinterpret_cast<const float4*>(D.lights), i);
            const float d2 = box_d2(E.ex, E.ey, E.ez, P.x, P.y, P.z, P.x, P.y, P.z);
            emit = rr_test(rotated(i, E.R), D, d2, true);
            if (W) w = 1.0f / accept_p(D.s, d2, 1.0f);
            ++tests;
        }
        emit2<W>(O, D, emit, make_uint2(E.u, i), w, false, make_uint2(0u, 0u), 0.0f);
    }
}

// Occupancy.  With one eye per wave the LDS holds 7 waves per SIMD (a wave
// takes its stack ring and the 4160-byte record area, 5696 bytes at the
// default 192 entries; 28 waves fill 160 KB), so the register budget is the
// one of 7 waves (72 VGPRs): asking for 8 only forced spills (frame
// 108.6 -> 108.3 ms with 7).  Several eyes per wave use little LDS and run
// at whatever occupancy their registers allow.
template <int EPW, int METHOD, bool STATS, bool W>
__global__ __launch_bounds__(kWave * kWavesPerBlock)
__attribute__((amdgpu_waves_per_eu(EPW == 1 ? 7 : 1, 8)))
void traverse_kernel(TravArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    // dynamic LDS: task table (n_items + 1 entries, padded to 16 bytes), then one area per wave
    uint32_t* task_begin_lds = reinterpret_cast<uint32_t*>(smem);
    for (uint32_t t = threadIdx.x; t <= A.n_items; t += blockDim.x) task_begin_lds[t] = A.task_begin[t];
    __syncthreads();
    unsigned char* wave_area = smem + (((size_t)A.n_items + 1u) * sizeof(uint32_t) + 15u) / 16u * 16u;

    const uint32_t lane = lane_id();
    const uint32_t wv = threadIdx.x / kWave;
    const uint32_t wave_gid = blockIdx.x * kWavesPerBlock + wv;
    const uint32_t cap = A.stack_cap;

    unsigned char* base = wave_area + (size_t)wv * A.lds_per_wave;
    WaveLds L;
    L.stack = reinterpret_cast<uint2*>(base);
    L.eyes = reinterpret_cast<uint32_t*>(base + (size_t)cap * sizeof(uint2));
    L.xpose = base + (size_t)cap * sizeof(uint2);   // one eye per wave: no eye table
    // the record area's LDS address, wave-uniform (the destination of the
    // record fetch must be a scalar)
    const uint32_t xlds = uni((uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)L.xpose);
    uint2* spill = reinterpret_cast<uint2*>(A.spill) + (size_t)wave_gid * A.spill_cap;

    uint64_t st_eyes = 0, st_visits = 0, st_rmq = 0, st_leaf = 0, st_spills = 0;
    uint32_t st_maxstack = 0;

    uint32_t cur = 0xFFFFFFFFu;
    ItemDesc D;
    OutState O;
    O.chunk = kNoChunk;
    O.wp = nullptr;
    O.ww = nullptr;
    O.fill = 0;
    O.count = 0;

    // work queues: start on this block's XCD queue, move on when it is empty
    uint32_t q = blockIdx.x % kQueues;
    uint32_t queues_left = kQueues;
    for (;;) {
        uint32_t i = 0;
        if (lane == 0) i = atomicAdd(A.queues + q * kQueueStride, 1u);
        i = uni(i);
        // the i-th task of queue q; increasing in i, so the first one past the
        // end means the queue is exhausted
        const uint32_t sh = A.interleave_shift;
        const uint64_t t64 = sh ? (((((uint64_t)(i >> sh)) * kQueues + q) << sh) | (i & ((1u << sh) - 1u)))
                                : (uint64_t)A.queue_begin[q] + i;
        const uint64_t end = sh ? (uint64_t)A.n_tasks : (uint64_t)A.queue_begin[q + 1];
        if (t64 >= end) {
            if (--queues_left == 0) break;
            q = (q + 1) % kQueues;
            continue;
        }
        const uint32_t t = (uint32_t)t64;

        // item of task t: largest k with task_begin[k] <= t
        uint32_t lo = 0, hi = A.n_items;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (task_begin_lds[mid] <= t) lo = mid; else hi = mid;
        }
        const uint32_t it = uni(lo);
        if (it != cur) {
            if (cur != 0xFFFFFFFFu) close_item(O, D, A.error);
            cur = it;
            D = A.items[it];
        }
        const uint32_t u0 = (t - D.task_begin) * EPW;
        const uint32_t cnt = min((uint32_t)EPW, D.n_virtual - u0);
        const uint32_t N = D.n_lights;
        const uint32_t leaf = D.leaf_size;
        const float s = D.s;

        // -------- eyes of this task --------
        EyeState E0;   // EPW == 1: wave-uniform eye
        if (EPW == 1) {
            const uint32_t u = D.order ? uni(D.order[u0]) : u0;
            E0 = load_eye(D, A.tile, u);
            E0.ex = unif(E0.ex); E0.ey = unif(E0.ey); E0.ez = unif(E0.ez);
            E0.R = uni(E0.R); E0.kr = uni(E0.kr);
        } else {
            if (lane < cnt) {
                const uint32_t u = D.order ? D.order[u0 + lane] : u0 + lane;
                const EyeState e = load_eye(D, A.tile, u);
                uint32_t* w = L.eyes + lane * 8u;
                w[0] = __float_as_uint(e.ex); w[1] = __float_as_uint(e.ey); w[2] = __float_as_uint(e.ez);
                w[3] = e.R; w[4] = e.kr; w[5] = e.u;
            }
            wave_sync();
        }
        if (STATS) st_eyes += cnt;

        StackState S;
        S.g = 0; S.n = 0; S.base = 0; S.max_total = 0; S.spills = 0;

        // -------- roots --------
        {
            const bool act = lane < cnt;
            EyeState E = E0;
            if (EPW > 1 && act) {
                const uint32_t* w = L.eyes + lane * 8u;
                E.ex = __uint_as_float(w[0]); E.ey = __uint_as_float(w[1]); E.ez = __uint_as_float(w[2]);
                E.R = w[3]; E.kr = w[4]; E.u = w[5];
            }
            if (D.n_nodes == 0) {
                // the whole light set is one leaf: exact tests of its <= 8 lights
                uint64_t tests = 0;
                if (EPW == 1) {
                    // spread the lights of the single eye over the lanes
                    const bool a1 = lane < N;
                    bool emit = false;
                    float w = 0.0f;
                    if (a1) {
                        const float4 P = load_global4(reinterpret_cast<const float4*>(D.lights), lane);
                        const float d2 = box_d2(E.ex, E.ey, E.ez, P.x, P.y, P.z, P.x, P.y, P.z);
                        emit = rr_test(rotated(lane, E.R), D, d2, true);
                        if (W) w = 1.0f / accept_p(s, d2, 1.0f);
                        ++tests;
                    }
                    emit2<W>(O, D, emit, make_uint2(E.u, lane), w, false, make_uint2(0u, 0u), 0.0f);
                } else {
                    leaf_lights<W>(O, D, E, 0u, act ? N : 0u, 0u, 0u, tests);
                }
                if (STATS) st_leaf += tests;
                continue;
            }
            if (EPW == 1 && D.n_frontier > 0) {
                // one eye per wave: lane t tests entry t of the hierarchy's top
                // (its range minimum, its box; a leaf entry is tested as a leaf
                // child is), surviving nodes are pushed in index order
                const bool fa = lane < D.n_frontier;
                uint32_t a = 0, b = 1, rec = 0xFFFFFFFFu;
                float4 f0 = make_float4(0.f, 0.f, 0.f, 0.f), f1 = f0;
                if (fa) {
                    const float4* f = reinterpret_cast<const float4*>(D.frontier) + 3u * lane;
                    f0 = f[0];
                    f1 = f[1];
                    a = __float_as_uint(f0.w);
                    b = __float_as_uint(f1.w);
                    rec = __float_as_uint(f[2].x);
                }
                const uint32_t n = b - a;
                uint32_t k = a;
                if (METHOD == 0 || METHOD == 5) {
                    k = rmq<METHOD>(a, b, E.kr);   // a one-index range gives a
                } else if (n > 1u) {
                    k = rmq<METHOD>(a, b, E.kr);
                }
                if (STATS && fa && n > 1u) ++st_rmq;
                const uint32_t v = rotated(k, E.R);
                const float d2 = box_d2(E.ex, E.ey, E.ez, f0.x, f0.y, f0.z, f1.x, f1.y, f1.z);
                bool kept = false;
                if (fa) kept = rr_test(v, D, d2, n == 1u);
                const bool push = kept && rec != 0xFFFFFFFFu;
                const bool emit = kept && rec == 0xFFFFFFFFu && n == 1u;
                const bool multi = kept && rec == 0xFFFFFFFFu && n > 1u;
                float w = 0.0f;
                if (W && emit) w = 1.0f / accept_p(s, d2, 1.0f);
                const uint64_t m = ballot(push);
                if (push) L.stack[count_below(m)] = make_uint2(rec, k);
                S.n = (uint32_t)__popcll(m);
                wave_sync();
                // each pair of entries is one parent's two child tests
                if (STATS) st_visits += (D.n_frontier + 1u) / 2u;
                emit2<W>(O, D, emit, make_uint2(E.u, a), w, false, make_uint2(0u, 0u), 0.0f);
                if (ballot(multi)) {
                    uint64_t tests = 0;
                    leaf_lights<W>(O, D, E, a, multi ? n : 0u, 0u, 0u, tests);
                    if (STATS) st_leaf += tests;
                }
            } else {
            bool push = false;
            uint32_t k0 = 0;
            if (act) {
                k0 = rmq<METHOD>(0u, N, E.kr);
                const float d2 = box_d2(E.ex, E.ey, E.ez, D.root_lo[0], D.root_lo[1], D.root_lo[2],
                                        D.root_hi[0], D.root_hi[1], D.root_hi[2]);
                push = rr_test(rotated(k0, E.R), D, d2, false);
                if (STATS) ++st_rmq;
            }
            const uint64_t m = ballot(push);
            if (push) {
                const uint32_t at = count_below(m);
                L.stack[at] = make_uint2(0u | ((EPW > 1 ? lane : 0u) << kSlotShift), k0);
            }
            S.n = (uint32_t)__popcll(m);
            wave_sync();
            }
        }

        // -------- top-down walk --------
        // the node records' base, wave-uniform in scalar registers for the
        // whole walk (the loads take it as their scalar base)
        const Node* const nodes = reinterpret_cast<const Node*>(uni64((unsigned long long)(size_t)D.nodes));
        // the loop and refill conditions are written as one scalar compare
        // each (S.g is a multiple of 64, so S.n < 64 && S.g > 0 is
        // S.n < min(S.g, 64)); as && / + the compiler builds them from two
        // compares merged in lane masks
        while ((S.n | S.g) != 0u) {
            if (S.n < min(S.g, (uint32_t)kStackUnit)) stack_refill(S, L, spill, cap);
            // the wave issues its record loads at raised priority, so that
            // they leave early (frame 142.9 -> 142.1 ms)
            __builtin_amdgcn_s_setprio(1);
            const uint32_t n = min(S.n, (uint32_t)kWave);
            const bool act = lane < n;
            // inactive lanes keep an arbitrary entry: every load and decision
            // below is masked by `act` (no instruction spent on a default)
            uint2 e;
            e.x = __builtin_nondeterministic_value(e.x);
            e.y = __builtin_nondeterministic_value(e.y);
            if (act) e = L.stack[ring(S.base + S.n - n + lane, cap)];
            S.n -= n;
            wave_sync();
            if (STATS) st_visits += n;

            EyeState E = E0;
            const uint32_t node = e.x & (kMaxNodes - 1u);
            const uint32_t slot = e.x >> kSlotShift;
            if (EPW > 1 && act) {
                const uint32_t* w = L.eyes + slot * 8u;
                E.ex = __uint_as_float(w[0]); E.ey = __uint_as_float(w[1]); E.ez = __uint_as_float(w[2]);
                E.R = w[3]; E.kr = w[4]; E.u = w[5];
            }

            bool pushL = false, pushR = false, emitL = false, emitR = false, multi = false;
            // read only in lanes whose flags above are set
            uint32_t kL = __builtin_nondeterministic_value(kL), kR = __builtin_nondeterministic_value(kR);
            uint32_t a = __builtin_nondeterministic_value(a), c = __builtin_nondeterministic_value(c);
            uint32_t b = __builtin_nondeterministic_value(b);
            uint32_t first = __builtin_nondeterministic_value(first);
            float wL = __builtin_nondeterministic_value(wL), wR = __builtin_nondeterministic_value(wR);
            uint32_t mlN = 0, mrN = 0;   // lights of the multi-light leaves to test (0: none)
            // Node records.  A load costs about one cycle of the vector-memory
            // pipeline per distinct cache line that a quad of lanes touches
            // (more when the line comes from L2 or beyond), so neighbouring
            // lanes share each record's line (see FetchOf).
            float4 q0, q1, q2, q3;
            if (FetchOf<EPW>::quad_lds) {
                // lane 4g + j fetches quarter j of the records of lanes 4g + t;
                // quarter j of record t lands at t * kSlab + 64 g + 16 j.
                // Inactive lanes fetch record 0, so no load needs a lane mask;
                // byte offsets are 32-bit (at most 2^26 records), the
                // base and the LDS destinations are wave-uniform.
                const uint32_t j = lane & 3u, g4 = lane & ~3u;
                const uint32_t nd = act ? node : 0u;
                const uint32_t jo = j << 4;
                const uint32_t o0 = ((uint32_t)__builtin_amdgcn_mov_dpp((int)nd, 0x00, 0xF, 0xF, false) << 6) | jo;
                const uint32_t o1 = ((uint32_t)__builtin_amdgcn_mov_dpp((int)nd, 0x55, 0xF, 0xF, false) << 6) | jo;
                const uint32_t o2 = ((uint32_t)__builtin_amdgcn_mov_dpp((int)nd, 0xAA, 0xF, 0xF, false) << 6) | jo;
                const uint32_t o3 = ((uint32_t)__builtin_amdgcn_mov_dpp((int)nd, 0xFF, 0xF, 0xF, false) << 6) | jo;
                typedef __attribute__((address_space(1))) const unsigned char* gbytes;
                typedef __attribute__((address_space(1))) const void* gptr;
                typedef __attribute__((address_space(3))) void* lptr;
                const gbytes rec = (gbytes)(nodes);
                __builtin_amdgcn_global_load_lds((gptr)(rec + o0), (lptr)(size_t)(xlds), 16, 0, 0);
                __builtin_amdgcn_global_load_lds((gptr)(rec + o1), (lptr)(size_t)(xlds + kSlab), 16, 0, 0);
                __builtin_amdgcn_global_load_lds((gptr)(rec + o2), (lptr)(size_t)(xlds + 2 * kSlab), 16, 0, 0);
                __builtin_amdgcn_global_load_lds((gptr)(rec + o3), (lptr)(size_t)(xlds + 3 * kSlab), 16, 0, 0);
                unsigned char* xb = L.xpose;
                __builtin_amdgcn_s_setprio(0);
                wave_sync();
                const float4* r = reinterpret_cast<const float4*>(xb + j * kSlab + 16u * g4);
                q0 = r[0]; q1 = r[1]; q2 = r[2]; q3 = r[3];
                wave_sync();
            } else {
                const bool odd = (lane & 1u) != 0u;
                const uint32_t partner = (uint32_t)__builtin_amdgcn_mov_dpp((int)node, kDppSwapPairs, 0xF, 0xF, false);
                const uint32_t n_even = odd ? partner : node;   // record of the pair's even lane
                const uint32_t n_odd = odd ? node : partner;    // record of the pair's odd lane
                const float4* re = reinterpret_cast<const float4*>(D.nodes + n_even);
                const float4* ro = reinterpret_cast<const float4*>(D.nodes + n_odd);
                const uint32_t h = odd ? 1u : 0u;
                float4 e02 = make_float4(0.f, 0.f, 0.f, 0.f), e13 = e02, o02 = e02, o13 = e02;
                if ((lane & ~1u) < n) { e02 = load_global4(re, h); e13 = load_global4(re, 2u + h); }
                if ((lane | 1u) < n) { o02 = load_global4(ro, h); o13 = load_global4(ro, 2u + h); }
                __builtin_amdgcn_s_setprio(0);
                // even lane holds chunks 0, 2 of both records, odd lane chunks 1, 3
                const float4 r1 = swap_pairs(odd ? e02 : o02);
                const float4 r2 = swap_pairs(odd ? e13 : o13);
                q0 = odd ? r1 : e02;
                q1 = odd ? o02 : r1;
                q2 = odd ? r2 : e13;
                q3 = odd ? o13 : r2;
            }
            // Every lane runs the node arithmetic (inactive ones on whatever
            // their registers hold, with no range-minimum query); only the
            // decisions are masked by `act`.  A block masked by `act` cost the
            // moves that merge its results with defaults every step, and spills
            // (frame 124.6 -> 122.8 ms).
            {
                a = __float_as_uint(q0.w);
                c = __float_as_uint(q1.w);
                b = __float_as_uint(q2.w);
                first = __float_as_uint(q3.w);
                const uint32_t k = e.y;
                // the child holding k inherits the minimum; the other one needs a query
                const bool kLeft = k < c;
                const uint32_t qa = kLeft ? c : a;
                uint32_t kq = qa;
                if (METHOD == 0 || METHOD == 5) {
                    // the default method returns qa for a one-index range, so
                    // it runs on every lane (inactive ones on [qa, qa + 1))
                    // without a divergent guard
                    const uint32_t qb = act ? (kLeft ? b : c) : qa + 1u;
                    kq = rmq<METHOD>(qa, qb, E.kr);
                    if (STATS && qb - qa > 1u) ++st_rmq;
                } else {
                    const uint32_t qb = act ? (kLeft ? b : c) : qa;
                    if (qb - qa > 1u) {
                        kq = rmq<METHOD>(qa, qb, E.kr);
                        if (STATS) ++st_rmq;
                    }
                }
                kL = kLeft ? k : kq;
                kR = kLeft ? kq : k;
                if (METHOD == 5) {   // ablation: the inheriting child's minimum is recomputed too
                    const uint32_t ia = kLeft ? a : c, ib = act ? (kLeft ? c : b) : ia;
                    uint32_t ki = ia;
                    if (ib - ia > 1u) {
                        ki = rmq<METHOD>(ia, ib, E.kr);
                        if (STATS) ++st_rmq;
                    }
                    kL = kLeft ? ki : kL;
                    kR = kLeft ? kR : ki;
                }
                const uint32_t nL = c - a, nR = b - c;
                const bool leafL = nL <= leaf, leafR = nR <= leaf;
                const float d2L = box_d2(E.ex, E.ey, E.ez, q0.x, q0.y, q0.z, q1.x, q1.y, q1.z);
                const float d2R = box_d2(E.ex, E.ey, E.ez, q2.x, q2.y, q2.z, q3.x, q3.y, q3.z);
                const uint32_t vL = rotated(kL, E.R), vR = rotated(kR, E.R);
                bool sL, sR;
                const bool openL = rr_fast(vL, D, d2L, nL == 1u, sL) && act;
                const bool openR = rr_fast(vR, D, d2R, nR == 1u, sR) && act;
                if (openL || openR) {   // rare: one shared block for the IEEE decisions
                    if (openL) sL = keeps(vL, accept_p(s, d2L, nL == 1u ? 1.0f : kBoxMargin));
                    if (openR) sR = keeps(vR, accept_p(s, d2R, nR == 1u ? 1.0f : kBoxMargin));
                }
                sL = sL && act;
                sR = sR && act;
                pushL = sL && !leafL;
                pushR = sR && !leafR;
                emitL = sL && nL == 1u;
                emitR = sR && nR == 1u;
                if (W) {
                    if (emitL) wL = 1.0f / accept_p(s, d2L, 1.0f);
                    if (emitR) wR = 1.0f / accept_p(s, d2R, 1.0f);
                }
                mlN = sL && leafL && nL > 1u ? nL : 0u;
                mrN = sR && leafR && nR > 1u ? nR : 0u;
                multi = mlN + mrN > 0u;
            }

            // push survivors: a lane's two children stay adjacent, lanes in order
            const uint64_t bl = ballot(pushL), br = ballot(pushR);
            const uint32_t npush = (uint32_t)(__popcll(bl) + __popcll(br));
            if (npush) {
                if (S.n + npush > cap) {
                    if (!stack_spill(S, L, spill, cap, A.spill_cap, A.error)) break;
                }
                // S.n + npush <= cap here, so S.base + at < 2 cap
                const uint32_t at = S.n + count_below(bl) + count_below(br);
                const uint32_t tag = (EPW > 1 ? slot : 0u) << kSlotShift;
                if (pushL) L.stack[ring(S.base + at, cap)] = make_uint2(first | tag, kL);
                if (pushR) L.stack[ring(S.base + at + (pushL ? 1u : 0u), cap)] = make_uint2((first + 1u) | tag, kR);
                S.n += npush;
                wave_sync();
                const uint32_t tot = S.g + S.n;
                if (tot > S.max_total) S.max_total = tot;
            }

            // one-light leaves accepted at the parent
            emit2<W>(O, D, emitL, make_uint2(E.u, a), wL, emitR, make_uint2(E.u, c), wR);

            // multi-light leaves
            if (leaf > 1u && ballot(multi)) {   // one-light leaves are emitted above
                uint64_t tests = 0;
                leaf_lights<W>(O, D, E, a, mlN, c, mrN, tests);
                if (STATS) st_leaf += tests;
            }
        }
        if (STATS) {
            st_spills += S.spills;
            st_maxstack = max(st_maxstack, S.max_total);
        }
    }
    if (cur != 0xFFFFFFFFu) close_item(O, D, A.error);

    if (STATS && A.stats) {
        uint64_t v[6] = {st_eyes, 0, st_visits, st_rmq, st_leaf, st_spills};
        for (int q = 0; q < 6; ++q) {
            uint64_t x = v[q];
            for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
            v[q] = x;
        }
        uint32_t mx = st_maxstack;
        for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor(mx, o));
        if (lane == 0) {
            // eyes / visits / spills / max stack are per-wave quantities kept in every lane
            atomicAdd(A.stats + ST_EYES, (unsigned long long)(v[0] / kWave));
            atomicAdd(A.stats + ST_VISITS, (unsigned long long)(v[2] / kWave));
            atomicAdd(A.stats + ST_RMQ, (unsigned long long)v[3]);
            atomicAdd(A.stats + ST_LEAF, (unsigned long long)v[4]);
            atomicAdd(A.stats + ST_SPILLS, (unsigned long long)(v[5] / kWave));
            atomicMax(A.stats + ST_MAXSTACK, (unsigned long long)mx);
        }
    }
}

// ---------------------------------------------------------------------------
// block walk: the default traversal
// ---------------------------------------------------------------------------
//
// In an aligned block [p, p + 2^v) of sequence indices the random numbers are
// evenly spaced: bitreverse(p + q) = bitreverse(p) + bitreverse_v(q)
// 2^(32-v), so with u = bitreverse(p) + R (mod 2^32) the index whose low bits
// are the reversal of x, x = -(u div 2^(32-v)) + t (mod 2^v), has the value
// (u mod 2^(32-v)) + t 2^(32-v), t = 0, 1, ..., 2^v - 1.  The range minimum is
// the t = 0 member, and every index whose number passes a bound T comes next
// in closed form: a block's candidates are the first
//     1 + ((T - u mod 2^(32-v)) div 2^(32-v))
// members, none when the minimum fails.  So the walk does not have to descend
// to the lights.  It bounds a block's acceptance by the distance to its box,
// counts the candidates that pass the bound, and only splits a block while
// that bound is loose (many candidates would fail their own test); otherwise
// it lists the candidates, and each is tested exactly like a one-light leaf.
// On the 1920x1080 x 2^20 frame an eye's 2,342 accepted pairs take 1,285 box
// tests and 4,085 candidate tests (simulated for 3,001 of its eyes with the
// split rule below), where the node walk tests 25,500 children, each with a range
// minimum: 4,700 vector instructions an eye a wave, 20.1 ms a frame against
// 101.7 .. 106.6.  What bounds it: the L1's line accesses
// (1.0e10 a frame, 0.9 per CU-cycle; one per cycle is its rate), four fifths of
// them candidates' lights, one line per lane where neighbouring lanes do not
// share it; hence the eye order by shift class, and 16 eyes of that order to
// a step (below).
//
// One wave takes a task of up to 64 eyes of an item and keeps two LIFO lists
// in LDS.  `stack` holds split blocks (block number | eye slot << 26): a step
// pops up to 16 of them and every lane tests one child, lane 16 c + j child c
// of the j-th: 16 eyes that stand at the same block read one line, and their
// children are pushed child by child, so the 16 go on together (frame 38.8 ->
// 35.4 ms against four adjacent lanes to a parent).  `queue` holds candidates
// (light | eye slot << 26, bit-reversed: a block's candidates are 2^(32-v)
// apart in that form, and one add from their random numbers): whenever it holds
// 64 they are tested, one per lane.  Accepted pairs wait in LDS and leave 64 at
// a time, in whole cache lines (35.4 -> 27.5 ms together with the listing by
// prefix sums: 38.0 instead of 41.5 GB written).  Eyes enter one root at a time
// as the stack drains, so both kinds of step run full lanes also where an eye
// has little work.  Lanes read their eye (position, rotation) from LDS by slot.
// A lane's candidates stand next to each other in the queue: one candidate of
// every lane in turn instead, which would let eyes of one shift at one block
// read a light together, takes 25 ms a frame in any eye order against 19.
//
// Stack bound: a step pops 16 parents and pushes at most 64 children while the
// stack holds at most kCullWide entries, so it leaves at most kCullWide + 48;
// above kCullWide it pops one parent at a time, which adds at most 3 entries per
// level (at most 11 levels) until that parent's subtree is done.
constexpr uint32_t kCullStack = 256;
constexpr uint32_t kCullWide = 160;       // entries above which parents are popped one at a time
constexpr uint32_t kCullQueue = 384;      // at least 64 + 16 (see the listing rounds)
constexpr uint32_t kCullStage = 2 * kWave;        // staged pairs: chunked output
constexpr uint32_t kCullStageDense = 8 * kWave;   // ... dense output (see DENSE)
constexpr uint32_t kCullSlotShift = 26;   // block numbers are below 2^23, lights below 2^25
constexpr uint32_t kCullEyes = kWave;     // eye slots of a wave
constexpr uint32_t cull_wave_bytes(bool weights, bool dense) {
    return kCullEyes * 16 + kCullStack * 4 + kCullQueue * 4 + kCullEyes * 4 +
           (dense ? kCullStageDense : kCullStage) * (weights ? 12u : 8u);
}
// A block is split while the candidates that its bound lets through beyond
// those that must be near enough, cnt * (1 - far bound / near bound), exceed
// kCullWaste (cost of four more box tests against that of the candidates they
// save), or while there are more than kCullMaxRun of them (a lane lists its
// candidates one per turn).  Measured, full frame / quarter frame / batch of 64
// caches, ms: 4: 22.2 / 7.30 / 3.34, 6: 21.3 / 7.06 / 3.37, 8: 21.0 / 6.95 /
// 3.44, 12: 21.05 / - / -; runs of 8, 16, 32 at the frame: 21.6, 21.1, 21.3.
constexpr float kCullWaste = 6.0f;
constexpr uint32_t kCullMaxRun = 16;

struct CullLds {
    uint32_t* stack;
    uint32_t* queue;
    float4* eyes;      // x, y, z, bits of R less the reversed tree and slot bits:
                       // a reversed queue entry plus this is the rotated inverse
    uint32_t* u;       // virtual eye index
    uint2* pairs;      // accepted pairs waiting to be stored
    float* d2;         // their squared distances (weights are computed as pairs are stored)
};

// The item's descriptor through the constant address space: no kernel of the
// launch writes it, so its fields come by scalar loads into scalar registers
// (from the generic address the compiler loads them into vector registers and
// reads them back lane by lane: two or three instructions per use and step).
// The address is opaque to the compiler: each caller loads the fields it uses
// where it uses them, and the walk's inner loops hold only their own (all of an
// item's fields held across the loops spill scalar registers to vector lanes).
__device__ __forceinline__ void load_item(ItemDesc& D, const ItemDesc* p) {
    typedef const __attribute__((address_space(4))) uint32_t* cptr;
    unsigned long long at = uni64((unsigned long long)(size_t)p);
    asm volatile("" : "+s"(at));
    const cptr src = (cptr)at;
    uint32_t w[sizeof(ItemDesc) / 4];
    static_assert(sizeof(ItemDesc) % 4 == 0, "whole words");
#pragma unroll
    for (uint32_t q = 0; q < sizeof(ItemDesc) / 4; ++q) w[q] = src[q];
    __builtin_memcpy(&D, w, sizeof D);
}

// 16 bytes at a 32-bit byte offset from a uniform base.
__device__ __forceinline__ float4 load_at(const float4* base, uint32_t offset) {
    typedef const __attribute__((address_space(1))) unsigned char* gbytes;
    const f32x4 v = *(const __attribute__((address_space(1))) f32x4*)((gbytes)(base) + offset);
    return make_float4(v.x, v.y, v.z, v.w);
}

// The larger of two floats that are not negative, by their bits (the float
// maximum costs one more instruction, which quiets a signalling b).
__device__ __forceinline__ float max_bits(float a, float b) {
    return __uint_as_float(max(__float_as_uint(a), __float_as_uint(b)));
}

// The smaller of two floats, without the instructions that quiet a signalling
// NaN first (results of arithmetic are none; the compiler no longer knows where
// they come from another basic block).
__device__ __forceinline__ float min_plain(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// x >= 0 to u32, rounded down, saturating (a C++ conversion leaves the result
// past 2^32 undefined; the instruction saturates).
__device__ __forceinline__ uint32_t to_u32_sat(float x) {
    uint32_t r;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// Inclusive sum over the wave's lanes (DPP row shifts, then row broadcasts).
__device__ __forceinline__ uint32_t wave_sum_inclusive(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
    asm("" : "+v"(x));   // or `sum - c` takes the last additions apart, two instructions each
    return x;
}

// Take a chunk: as alloc_chunk and set_chunk, with the two buffers' addresses in
// scalar registers (a select between two fields of a descriptor goes through
// scratch memory).
template <bool W>
__device__ __forceinline__ void cull_open(OutState& O, const ItemDesc* item) {
    ItemDesc D;
    load_item(D, item);
    const unsigned long long pairs = uni64((unsigned long long)(size_t)D.pairs);
    const unsigned long long slack_pairs = uni64((unsigned long long)(size_t)D.slack_pairs);
    const unsigned long long weights = W ? uni64((unsigned long long)(size_t)D.weights) : 0ull;
    const unsigned long long slack_weights = W ? uni64((unsigned long long)(size_t)D.slack_weights) : 0ull;
    O.chunk = alloc_chunk(D);
    O.fill = 0;
    const unsigned long long p0 = O.chunk << D.chunk_shift, C = 1ull << D.chunk_shift;
    const unsigned long long q0 = p0 - D.capacity;
    unsigned long long wp = 0, ww = 0;
    if (p0 + C <= D.capacity) {
        wp = pairs + p0 * 8u;
        ww = weights + p0 * 4u;
    } else if (p0 >= D.capacity && q0 + C <= D.slack) {
        wp = slack_pairs + q0 * 8u;
        ww = slack_weights + q0 * 4u;
    }
    O.wp = reinterpret_cast<uint2*>(uni64(wp));
    if (W) O.ww = reinterpret_cast<float*>(uni64(ww));
}

// Store the newest n (1 .. 64) staged pairs, [end - n, end): into the wave's
// chunk, at O.fill, which is a multiple of 64 here.  Chunks hold a multiple of
// 64, so a run never crosses one, and whole runs are whole cache lines.
template <bool W>
__device__ __forceinline__ void cull_store(OutState& O, const ItemDesc* item, uint32_t chunk_shift, float s,
                                           const CullLds& L, uint32_t end, uint32_t n) {
    const uint32_t lane = lane_id();
    wave_sync();
    if (O.chunk == kNoChunk) {
        cull_open<W>(O, item);
    }
    if (lane < n) {
        const uint2 pr = L.pairs[end - n + lane];
        const float w = W ? 1.0f / accept_p(s, L.d2[end - n + lane], 1.0f) : 0.0f;
        if (O.wp) {
            put_pair(O.wp, O.fill + lane, pr);
            if (W) put_weight(O.ww, O.fill + lane, w);
        } else {   // a chunk across the capacity or past the slack
            ItemDesc D;
            load_item(D, item);
            store_pair<W>(D, (O.chunk << chunk_shift) + O.fill + lane, pr, w);
        }
    }
    O.fill += n;
    O.count += n;
    if (O.fill >> chunk_shift) {
        O.chunk = kNoChunk;
        O.wp = nullptr;
    }
}

// Dense output: the n staged pairs go to positions [base, base + n).
template <bool W>
__device__ __forceinline__ void cull_store_at(const ItemDesc& D, const CullLds& L, unsigned long long base, uint32_t n) {
    wave_sync();
    for (uint32_t k = lane_id(); k < n; k += (uint32_t)kWave) {
        const unsigned long long at = base + k;
        if (at >= D.capacity) break;
        put_pair(reinterpret_cast<uint2*>(D.pairs), at, L.pairs[k]);
        if (W) put_weight(D.weights, at, 1.0f / accept_p(D.s, L.d2[k], 1.0f));
    }
    wave_sync();
}

// Dense output: the next n positions of the item.
__device__ __forceinline__ unsigned long long take_positions(const ItemDesc& D, unsigned long long n) {
    unsigned long long base = 0;
    if (lane_id() == 0) base = atomicAdd(D.counters + CNT_PAIRS, n);
    return uni64(base);
}

// Exact tests of the n (1 .. 64) newest candidates of the queue, which ends at
// entry `end`, one per lane; `staged` counts the pairs waiting in LDS.
template <bool W, bool DENSE>
__device__ __forceinline__ void cull_test(OutState& O, const ItemDesc& D, const ItemDesc* item, const CullLds& L,
                                          uint32_t end, uint32_t n, uint32_t& staged) {
    const uint32_t lane = lane_id();
    wave_sync();
    // n < 64 only where the queue holds no more (end == n), so every lane reads
    // inside it; what lanes past n read is any light and slot (the index is
    // clamped, the slot has 6 bits), and only their decision is masked
    const uint32_t r = L.queue[end - n + lane];
    const uint32_t c = bit_reverse(r), slot = c >> kCullSlotShift;
    const uint32_t i = c & ((1u << D.block_log) - 1u);
    // the light's place: the low bits of its index reversed (see
    // block_tree_lights; 1.07e10 -> 9.8e9 line accesses a frame, 19.5 -> 19.3 ms,
    // batch of 64 caches 3.30 -> 3.14 ms)
    const uint32_t leaf_log = block_leaf_log(D.block_log);
    const uint32_t place = (i & (0u - (1u << leaf_log))) | r >> (32u - leaf_log);
    const uint32_t last = (D.n_lights - 1u) | ((1u << leaf_log) - 1u);
    const float4 P = load_at(reinterpret_cast<const float4*>(D.lights), min(place, last) << 4);
    const float4 e = L.eyes[slot];
    const float dx = P.x - e.x, dy = P.y - e.y, dz = P.z - e.z;
    const float x2 = dx * dx, y2 = dy * dy, z2 = dz * dz;
    float d2 = (x2 + y2) + z2;
    const uint32_t v = r + __float_as_uint(e.w);   // the rotated inverse (see CullLds)
    // the product-form test (see rr_test) as lane masks
    const float prod = (float)v * d2;
    const uint64_t near = ballot(d2 <= D.d2_fast);   // not where d2 is NaN
    const uint64_t sure = ballot(prod < D.t_keep) & near;
    const uint64_t cull = ballot(prod > D.t_cull) & near;
    const uint64_t valid = ballot(i < D.n_lights) & (~0ull >> (64u - n));
    uint64_t m = sure & valid;
    const uint64_t open = valid & ~(sure | cull);
    if (open) {   // rare: the IEEE decision
        bool keep = false;
        if (__builtin_amdgcn_inverse_ballot_w64(open)) {
            // |l - e| per axis, 0 where it is NaN: box_d2 of a one-point box
            const float ax = fmaxf(fabsf(dx), 0.0f), ay = fmaxf(fabsf(dy), 0.0f), az = fmaxf(fabsf(dz), 0.0f);
            const float ax2 = ax * ax, ay2 = ay * ay, az2 = az * az;
            d2 = (ax2 + ay2) + az2;
            keep = keeps(v, accept_p(D.s, d2, 1.0f));
        }
        m |= ballot(keep);
    }
    if (D.capacity == 0) {   // counting launch: nothing is stored
        O.count += (uint32_t)__popcll(m);
        return;
    }
    if (__builtin_amdgcn_inverse_ballot_w64(m)) {
        const uint32_t at = staged + count_below(m);
        L.pairs[at] = make_uint2(L.u[slot], i);
        if (W) L.d2[at] = d2;
    }
    staged += (uint32_t)__popcll(m);
    if (DENSE) {
        if (staged > kCullStageDense - (uint32_t)kWave) {   // no room for another test's pairs
            ItemDesc X;
            load_item(X, item);
            cull_store_at<W>(X, L, take_positions(X, staged), staged);
            staged = 0;
        }
    } else if (staged >= (uint32_t)kWave) {
        cull_store<W>(O, item, D.chunk_shift, D.s, L, staged, kWave);
        staged -= kWave;
    }
}

// A wave leaves an item: its last staged pairs, then close_item.
template <bool W, bool DENSE>
__device__ __forceinline__ void cull_close(OutState& O, const ItemDesc* item, const CullLds& L, uint32_t& staged,
                                           uint32_t* err) {
    ItemDesc D;
    load_item(D, item);
    if (DENSE) {
        const unsigned long long n = D.capacity ? staged : O.count;
        if (n) {
            const unsigned long long base = take_positions(D, n);
            cull_store_at<W>(D, L, base, staged);
        }
        O.count = 0;
    } else {
        if (staged) cull_store<W>(O, item, D.chunk_shift, D.s, L, staged, staged);
        close_item(O, D, err);
    }
    staged = 0;
}

// DENSE: the output of launches with few pairs.  A wave stages up to 512 pairs
// and takes exactly as many positions with one atomic, so the output is dense
// as it is written and needs no chunks and no compaction; the last pairs of a
// block's four waves share one atomic.  Same-address atomics are the cost (about
// 13 ns each on this GPU): 512 staged pairs keep them below the cost of chunks
// and compaction up to about 2^24 pairs (block_walk_dense), and larger outputs
// take the chunks of thousands of pairs.
template <bool W, bool DENSE>
__global__ __launch_bounds__(kWave * kWavesPerBlock)
__attribute__((amdgpu_waves_per_eu(DENSE ? 1 : (W ? 7 : 8), 8)))
void cull_kernel(TravArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    // dynamic LDS: one area per wave, then the task table (n_items + 1 entries)
    uint32_t* task_begin_lds = reinterpret_cast<uint32_t*>(smem + kWavesPerBlock * cull_wave_bytes(W, DENSE));
    for (uint32_t t = threadIdx.x; t <= A.n_items; t += blockDim.x) task_begin_lds[t] = A.task_begin[t];
    __syncthreads();
    const uint32_t lane = lane_id();
    CullLds L;
    {
        unsigned char* base = smem + uni(threadIdx.x / kWave) * cull_wave_bytes(W, DENSE);
        L.eyes = reinterpret_cast<float4*>(base);
        L.pairs = reinterpret_cast<uint2*>(base + kCullEyes * 16);
        L.stack = reinterpret_cast<uint32_t*>(L.pairs + (DENSE ? kCullStageDense : kCullStage));
        L.queue = L.stack + kCullStack;
        L.u = L.queue + kCullQueue;
        L.d2 = reinterpret_cast<float*>(L.u + kCullEyes);   // with W only
    }
    uint32_t staged = 0;
    uint32_t cur = 0xFFFFFFFFu;
    OutState O;
    O.chunk = kNoChunk;
    O.wp = nullptr;
    O.ww = nullptr;
    O.fill = 0;
    O.count = 0;

    // work queues: start on this block's XCD queue, move on when it is empty
    uint32_t q = blockIdx.x % kQueues;
    uint32_t queues_left = kQueues;
    for (;;) {
        uint64_t t64, end;
        if (DENSE && A.static_tasks) {
            t64 = queues_left == kQueues ? blockIdx.x * kWavesPerBlock + threadIdx.x / kWave : A.n_tasks;
            t64 = uni64(t64);
            end = A.n_tasks;
            queues_left = 1;
        } else {
            // another block's queue is looked at before it is taken from: the
            // end of a launch would else be eight atomics of every wave, 13 ns
            // apart on each queue's line
            uint32_t* const head = A.queues + q * kQueueStride;
            uint32_t i = 0;
            end = A.queue_begin[q + 1];
            if (queues_left != kQueues) i = uni(__hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            if (i < (uint32_t)end - A.queue_begin[q]) {
                i = 0;
                if (lane == 0) i = atomicAdd(head, 1u);
                i = uni(i);
            }
            t64 = (uint64_t)A.queue_begin[q] + i;
        }
        uint32_t it = 0xFFFFFFFFu;   // no task left
        const uint32_t t = (uint32_t)t64;
        if (t64 >= end) {
            if (--queues_left != 0) {
                q = (q + 1) % kQueues;
                continue;
            }
        } else {
            uint32_t lo = 0, hi = A.n_items;
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (task_begin_lds[mid] <= t) lo = mid; else hi = mid;
            }
            it = uni(lo);
        }
        if (it != cur || it == 0xFFFFFFFFu) {   // a wave may get no task at all
            if (DENSE && it == 0xFFFFFFFFu) break;   // the block's waves close together, below
            if (cur != 0xFFFFFFFFu) cull_close<W, DENSE>(O, A.items + cur, L, staged, A.error);
            if (it == 0xFFFFFFFFu) break;
            cur = it;
        }
        ItemDesc D;
        load_item(D, A.items + it);
        const uint32_t part = t - D.task_begin;
        const uint32_t u0 = part >> D.sub_log << D.task_shift;
        const uint32_t root = (1u << D.sub_log) | (part & ((1u << D.sub_log) - 1u));
        const uint32_t cnt = min(1u << D.task_shift, D.n_virtual - u0);
        const uint32_t N = D.n_lights;
        const float s = D.s;
        const uint32_t S = D.block_log, leaf_log = block_leaf_log(S);

        if (lane < cnt) {
            const uint32_t u = D.order ? D.order[u0 + lane] : u0 + lane;
            const EyeState e = load_eye(D, A.tile, u);
            // block numbers and candidates carry the tree bit 2^S above their
            // index and the slot above that; R less the reversal of both takes
            // them out of every rotation
            L.eyes[lane] = make_float4(e.ex, e.ey, e.ez,
                                       __uint_as_float(e.R - (1u << (31u - S)) - bit_reverse(lane << kCullSlotShift)));
            L.u[lane] = e.u;
        }
        const float4* const blocks = reinterpret_cast<const float4*>(uni64((unsigned long long)(size_t)D.blocks));

        uint32_t next = 0, sn = 0, qn = 0;   // eyes started; stack and queue entries
        for (;;) {
            if (sn < 16u && next < cnt) {
                const uint32_t add = min(16u - sn, cnt - next);
                if (lane < add) L.stack[sn + lane] = root | ((next + lane) << kCullSlotShift);
                sn += add;
                next += add;
            }
            if (sn == 0u) break;
            wave_sync();
            const uint32_t g = sn > kCullWide ? 1u : min(16u, sn);
            sn -= g;
            const bool act = (lane & 15u) < g;
            const uint32_t ent = L.stack[sn + min(lane & 15u, g - 1u)];
            const uint32_t tag = ent & ~((1u << kCullSlotShift) - 1u);
            const uint32_t id = (ent << 2 | lane >> 4) & ((4u << kCullSlotShift) - 1u);
            uint32_t slot = ent >> kCullSlotShift;
            asm("" : "+v"(slot));   // or the shift to an address takes an `and`
            const float4 b0 = load_at(blocks, id << 5), b1 = load_at(blocks, (id << 5) + 16u);
            const float4 e = L.eyes[slot];

            // squared distances to the nearest and the farthest point of the box
            const float ax = b0.x - e.x, ay = b0.y - e.y, az = b0.z - e.z;
            const float bx = e.x - b1.x, by = e.y - b1.y, bz = e.z - b1.z;
            const float nx = fmaxf(fmaxf(ax, bx), 0.0f), ny = fmaxf(fmaxf(ay, by), 0.0f),
                        nz = fmaxf(fmaxf(az, bz), 0.0f);
            const float nx2 = nx * nx, ny2 = ny * ny, nz2 = nz * nz;
            const float dn = max_bits((nx2 + ny2) + nz2, s);
            // T, at least every light's threshold minus one: t_cull is s 2^32
            // (1 + 2^-18) or more, which covers the reciprocal's and the
            // products' rounding
            const uint32_t T = to_u32_sat(D.t_cull * __builtin_amdgcn_rcpf(dn));

            const uint32_t v = (uint32_t)__builtin_clz(id) + (S - 31u), rsh = 32u - v;   // 2^v indices
            const uint32_t p = id << v;                              // first index, and the tree bit
            const uint32_t u = bit_reverse(p | tag) + __float_as_uint(e.w);
            const uint32_t m0 = __builtin_amdgcn_ubfe(u, 0u, rsh);   // the block's minimum
            uint32_t c = act && m0 <= T ? ((T - m0) >> rsh) + 1u : 0u;
            // (a block that holds no light is infinitely far: T = 0 lists at most
            // the one index whose random number is 0, which lies past N)
            const uint64_t wide = ballot(c > 1u) & ballot(v > leaf_log);
            uint64_t ms = 0;
            if (wide) {
                // (to the far side, lo - e and e - hi are negative)
                const float fx = min_plain(ax, bx), fy = min_plain(ay, by), fz = min_plain(az, bz);
                const float df = max_bits((fx * fx + fy * fy) + fz * fz, s);
                ms = wide & (ballot(c > kCullMaxRun) | ~ballot((float)c * (df - dn) < kCullWaste * df));
                if (__builtin_amdgcn_inverse_ballot_w64(ms)) {
                    L.stack[sn + count_below(ms)] = id | tag;
                    c = 0;
                }
                sn += (uint32_t)__popcll(ms);
            }

            // List the candidates, as reversals: the first is m0 less e.w, and
            // the rotated inverses of the others are 2^rsh apart.  A lane's
            // start in the queue is its prefix sum.
            const uint32_t inc = wave_sum_inclusive(c);
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
            const uint32_t first = m0 - __float_as_uint(e.w);
            // with no step to come, the queue is drained
            const uint32_t least = sn == 0u && next == cnt ? 1u : (uint32_t)kWave;
            uint32_t done = 0;
            do {
                uint32_t upto = total, take = c;
                if (total - done > kCullQueue - qn) {
                    // lanes whose candidates do not fit wait for the next round
                    // (a lane lists at most 16, so every round takes some)
                    const uint64_t wait = ballot(inc - done > kCullQueue - qn) & ballot(c != 0u);
                    upto = (uint32_t)__builtin_amdgcn_readlane((int)(inc - c), (int)__builtin_ctzll(wait));
                    if (__builtin_amdgcn_inverse_ballot_w64(wait)) take = 0;
                }
                uint32_t* at = L.queue + (qn + (inc - c) - done);
                uint32_t* const at_end = at + take;
                for (uint32_t r = first; at != at_end; ++at) {
                    *at = r;
                    r += 1u << rsh;
                }
                c -= take;
                qn += upto - done;
                done = upto;
                while (qn >= least) {
                    const uint32_t n = min(qn, (uint32_t)kWave);
                    cull_test<W, DENSE>(O, D, A.items + cur, L, qn, n, staged);
                    qn -= n;
                }
            } while (done < total);
        }
        wave_sync();
    }
    if (DENSE) {
        // the block's last pairs (or counts): one atomic where its waves hold
        // the same item
        __shared__ unsigned long long sums[kWavesPerBlock];
        __shared__ uint32_t held[kWavesPerBlock];
        __shared__ unsigned long long first;
        const uint32_t wv = threadIdx.x / kWave;
        ItemDesc D;
        load_item(D, A.items + (cur == 0xFFFFFFFFu ? 0u : cur));
        const unsigned long long mine = cur == 0xFFFFFFFFu ? 0ull : (D.capacity ? staged : O.count);
        if (lane == 0) {
            sums[wv] = mine;
            held[wv] = mine ? cur : 0xFFFFFFFFu;
        }
        __syncthreads();
        unsigned long long before = 0, total = 0;
        uint32_t item = 0xFFFFFFFFu;
        bool same = true;
        for (uint32_t w = 0; w < (uint32_t)kWavesPerBlock; ++w) {
            if (held[w] == 0xFFFFFFFFu) continue;
            same = same && (item == 0xFFFFFFFFu || item == held[w]);
            item = held[w];
            if (w < wv) before += sums[w];
            total += sums[w];
        }
        if (same) {   // uniform over the block
            if (total && threadIdx.x == 0) first = atomicAdd(A.items[item].counters + CNT_PAIRS, total);
            __syncthreads();
            if (mine && D.capacity) cull_store_at<W>(D, L, uni64(first) + before, staged);
        } else if (mine) {
            cull_close<W, true>(O, A.items + cur, L, staged, A.error);
        }
    }
}

// ---- building the block tree ----
//
// block_leaf_kernel: one thread per smallest block (which also writes its lights
// in their second order; with neighbouring threads on neighbouring lights
// instead, 2^20 lights build in the same 0.79 ms), and in the same launch the
// four levels above it inside each thread block (256 blocks -> 64 -> 16 -> 4
// -> 1); block_up_kernel: the next four levels from a finished one.
struct BlockBox {
    float lo[3], hi[3];
};

__device__ __forceinline__ BlockBox empty_block() {
    BlockBox b;
    for (int k = 0; k < 3; ++k) {
        b.lo[k] = INFINITY;
        b.hi[k] = -INFINITY;
    }
    return b;
}

__device__ __forceinline__ void store_block(float4* blocks, uint32_t id, const BlockBox& b) {
    blocks[2u * id] = make_float4(b.lo[0], b.lo[1], b.lo[2], 0.0f);
    blocks[2u * id + 1u] = make_float4(b.hi[0], b.hi[1], b.hi[2], 0.0f);
}

// b: the box of block blockIdx.x * 256 + threadIdx.x of `level` (empty past its end)
__device__ __forceinline__ void block_levels(float4* blocks, uint32_t level, BlockBox b) {
    __shared__ BlockBox lds[256];
    const uint32_t t = threadIdx.x;
#pragma unroll 1
    for (uint32_t up = 1; up <= 4u && up <= level; ++up) {
        const uint32_t n = 256u >> (2u * up);
        if (t < 4u * n) lds[t] = b;
        __syncthreads();
        if (t < n) {
            b = lds[4u * t];
            for (uint32_t q = 1; q < 4u; ++q)
                for (int k = 0; k < 3; ++k) {
                    b.lo[k] = min_first(b.lo[k], lds[4u * t + q].lo[k]);
                    b.hi[k] = max_first(b.hi[k], lds[4u * t + q].hi[k]);
                }
            const uint32_t at = blockIdx.x * n + t, count = 1u << (2u * (level - up));
            if (at < count) store_block(blocks, count + at, b);
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void block_leaf_kernel(const float4* __restrict__ lights, uint32_t n_lights,
                                                         uint32_t block_log, float4* __restrict__ blocks,
                                                         float4* __restrict__ reversed) {
    const uint32_t leaf_log = block_leaf_log(block_log), level = (block_log - leaf_log) / 2u;
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    BlockBox b = empty_block();
    if (i < (1u << (2u * level))) {
        const uint64_t first = (uint64_t)i << leaf_log;
        for (uint32_t q = 0; q < (1u << leaf_log) && first < n_lights; ++q) {
            float4* const copy = reversed + first + (bit_reverse(q) >> (32u - leaf_log));
            if (first + q >= n_lights) {   // the last smallest block is filled up
                *copy = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                continue;
            }
            const float4 p = lights[first + q];
            *copy = p;
            b.lo[0] = min_first(b.lo[0], p.x); b.hi[0] = max_first(b.hi[0], p.x);
            b.lo[1] = min_first(b.lo[1], p.y); b.hi[1] = max_first(b.hi[1], p.y);
            b.lo[2] = min_first(b.lo[2], p.z); b.hi[2] = max_first(b.hi[2], p.z);
        }
        store_block(blocks, (1u << (2u * level)) + i, b);
    }
    block_levels(blocks, level, b);
}

__global__ __launch_bounds__(256) void block_up_kernel(uint32_t level, float4* __restrict__ blocks) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x, count = 1u << (2u * level);
    BlockBox b = empty_block();
    if (i < count) {
        const float4 lo = blocks[2u * (count + i)], hi = blocks[2u * (count + i) + 1u];
        b.lo[0] = lo.x; b.lo[1] = lo.y; b.lo[2] = lo.z;
        b.hi[0] = hi.x; b.hi[1] = hi.y; b.hi[2] = hi.z;
    }
    block_levels(blocks, level, b);
}

// ---------------------------------------------------------------------------
// the top of a hierarchy (the one-eye-per-wave walk's starting entries)
// ---------------------------------------------------------------------------
//
// One wave expands the root kFrontierDepth times: every internal entry is
// replaced by its two children (their boxes and ranges come from its record,
// their records are `first` and `first + 1` when internal), leaves stay.
// Entries keep index order; after level l there are at most 2^l of them.
// The root's own box is never needed: the root is internal (the caller only
// runs this for hierarchies with records) and is always expanded.
// A second block of the launch measures the spread of the lights' block tree
// (hrr_types.hpp) while the first one waits for its records.
__device__ __forceinline__ float block_spread(const float4* __restrict__ blocks, uint32_t n_lights) {
    const uint32_t log = block_tree_log(n_lights), leaf_log = block_leaf_log(log);
    const uint32_t n_blocks = ((n_lights - 1u) >> leaf_log) + 1u, first = 1u << (log - leaf_log);
    const uint32_t samples = min(n_blocks, kSpreadSamples);
    const float4 rlo = blocks[2], rhi = blocks[3];
    const float rl[3] = {rlo.x, rlo.y, rlo.z}, rh[3] = {rhi.x, rhi.y, rhi.z};
    float sum = 0.0f;
#pragma unroll   // the loads at once
    for (uint32_t r = 0; r < kSpreadSamples / 64u; ++r) {
        const uint32_t q = r * 64u + threadIdx.x;
        const uint32_t id = first + (uint32_t)((uint64_t)min(q, samples - 1u) * n_blocks / samples);
        const float4 lo = blocks[2u * id], hi = blocks[2u * id + 1u];
        const float l[3] = {lo.x, lo.y, lo.z}, h[3] = {hi.x, hi.y, hi.z};
        sum += q < samples ? block_share(l, h, rl, rh) : 0.0f;
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    return sum * ((float)n_blocks / (float)samples);
}

__global__ __launch_bounds__(64) void frontier_kernel(const Node* __restrict__ nodes, uint32_t n_lights,
                                                      uint32_t leaf, const float4* __restrict__ blocks,
                                                      float* __restrict__ out) {
    if (blockIdx.x == 1u) {
        const float spread = block_spread(blocks, n_lights);
        if (threadIdx.x == 0) out[kFrontierSpread] = spread;
        return;
    }
    struct Entry { uint32_t a, b, rec; float lo[3], hi[3]; };
    __shared__ Entry next[kFrontierMax];
    const uint32_t t = threadIdx.x;
    Entry e;
    e.a = 0u; e.b = n_lights; e.rec = 0u;
    for (int q = 0; q < 3; ++q) { e.lo[q] = 0.0f; e.hi[q] = 0.0f; }
    uint32_t n = 1;
    for (uint32_t level = 0; level < kFrontierDepth; ++level) {
        const bool have = t < n;
        const bool internal = have && e.rec != 0xFFFFFFFFu;
        const uint32_t c = have ? (internal ? 2u : 1u) : 0u;
        // exclusive prefix of c over the wave
        uint32_t inc = c;
        for (uint32_t off = 1; off < 64u; off <<= 1) {
            const uint32_t y = __shfl_up(inc, off, 64);
            if (t >= off) inc += y;
        }
        const uint32_t pos = inc - c;
        const uint32_t total = __shfl(inc, 63, 64);
        if (internal) {
            const Node R = nodes[e.rec];
            Entry L, Rt;
            L.a = R.a; L.b = R.c; L.rec = R.c - R.a > leaf ? R.first : 0xFFFFFFFFu;
            Rt.a = R.c; Rt.b = R.b; Rt.rec = R.b - R.c > leaf ? R.first + 1u : 0xFFFFFFFFu;
            for (int q = 0; q < 3; ++q) {
                L.lo[q] = R.lo_l[q]; L.hi[q] = R.hi_l[q];
                Rt.lo[q] = R.lo_r[q]; Rt.hi[q] = R.hi_r[q];
            }
            next[pos] = L;
            next[pos + 1u] = Rt;
        } else if (have) {
            next[pos] = e;
        }
        __syncthreads();
        n = total;
        if (t < n) e = next[t];
        __syncthreads();
    }
    if (t < n) {
        float* o = out + (size_t)t * kFrontierFloats;
        o[0] = e.lo[0]; o[1] = e.lo[1]; o[2] = e.lo[2]; o[3] = __uint_as_float(e.a);
        o[4] = e.hi[0]; o[5] = e.hi[1]; o[6] = e.hi[2]; o[7] = __uint_as_float(e.b);
        o[8] = __uint_as_float(e.rec); o[9] = 0.0f; o[10] = 0.0f; o[11] = 0.0f;
    }
    if (t == 0) reinterpret_cast<uint32_t*>(out)[kFrontierCount] = n;
}

// ---------------------------------------------------------------------------
// eye ordering: counting sort of the virtual eyes by (item, Morton cell, shift class)
// ---------------------------------------------------------------------------
//
// The traversal result does not depend on the order in which eyes are
// processed; processing spatially close eyes together lets an XCD's L2 hold
// the part of the hierarchy they share.  Cells: `bits` bits per axis of the
// eye position inside the item's light box, interleaved x-y-z.  Within a cell,
// eyes are grouped by the shift class: the low `rbits` significant bits of the
// eye's tile value t (t = m * 2^tz), bit reversed.  The minimum over an aligned
// block of 2^s indices is (bitreverse(p) + r) mod 2^(32-s), so two eyes whose
// m agree modulo 2^q see equal minima on every block with s >= 32 - tz - q;
// such eyes visit nearly the same nodes.  Bucket of virtual eye g of item k:
// ((k << 3 bits | cell) << rbits) | class.

__device__ __forceinline__ uint32_t spread3_10(uint32_t v) {
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ __forceinline__ uint32_t cell_of(float x, float lo, float scale, uint32_t bits) {
    const float f = (x - lo) * scale;
    const uint32_t top = (1u << bits) - 1u;
    if (!(f > 0.0f)) return 0u;
    const float c = floorf(f);
    return c >= (float)top ? top : (uint32_t)c;
}

__global__ __launch_bounds__(256) void order_keys_kernel(const OrderItem* __restrict__ items,
                                                         const uint32_t* __restrict__ vbegin, uint32_t n_items,
                                                         uint32_t total, uint32_t bits, uint32_t rbits,
                                                         const uint32_t* __restrict__ tile, uint32_t tile_tz,
                                                         uint32_t* __restrict__ keys, uint32_t* __restrict__ hist) {
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < total; g += gridDim.x * blockDim.x) {
        uint32_t lo = 0, hi = n_items;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (vbegin[mid] <= g) lo = mid; else hi = mid;
        }
        const OrderItem& I = items[lo];
        const uint32_t u = g - vbegin[lo];
        const uint32_t j = I.n_samples > 1 ? u / I.n_samples : u;
        const float* e = I.eyes + 3u * j;
        const uint32_t cx = cell_of(e[0], I.lo[0], I.scale[0], bits);
        const uint32_t cy = cell_of(e[1], I.lo[1], I.scale[1], bits);
        const uint32_t cz = cell_of(e[2], I.lo[2], I.scale[2], bits);
        uint32_t key = (lo << (3u * bits)) | (spread3_10(cx) << 2) | (spread3_10(cy) << 1) | spread3_10(cz);
        if (rbits) {
            const uint32_t pix = I.pixel_base + j;
            const uint32_t x = pix % I.width;
            const uint32_t y = pix / I.width;
            const uint32_t t = tile[(x & 63u) * 64u + (y & 63u)];
            key = (key << rbits) | (__brev(t >> tile_tz) >> (32u - rbits));
        }
        keys[g] = key;
        atomicAdd(hist + key, 1u);
    }
}

__global__ __launch_bounds__(256) void order_scatter_kernel(const uint32_t* __restrict__ keys,
                                                            const uint32_t* __restrict__ vbegin, uint32_t total,
                                                            uint32_t key_bits, uint32_t* __restrict__ offsets,
                                                            uint32_t* __restrict__ order) {
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < total; g += gridDim.x * blockDim.x) {
        const uint32_t key = keys[g];
        const uint32_t item = key >> key_bits;
        const uint32_t pos = atomicAdd(offsets + key, 1u);
        order[pos] = g - vbegin[item];
    }
}

// Output compaction after a traversal (the arithmetic and its bounds are in
// hrr_compact.hpp).  compact_plan_kernel, one block per item: the exclusive
// prefix sums of the hole lengths (partial-list order) and of the data
// lengths (chunk order) into the item's plan scratch, then the moved count,
// the dense count and the number of data chunks into its counter line.
// compact_move_kernel, a grid of blocks per item: moved element e goes from
// the e-th data position to the e-th hole position.

// Exclusive scan of one value per thread over a block of 256; total = the sum.
__device__ __forceinline__ unsigned long long block_exclusive_scan_u64(unsigned long long x,
                                                                       unsigned long long* lds,
                                                                       unsigned long long& total) {
    const uint32_t t = threadIdx.x;
    lds[t] = x;
    __syncthreads();
    for (uint32_t off = 1; off < 256u; off <<= 1) {
        const unsigned long long add = t >= off ? lds[t - off] : 0ull;
        __syncthreads();
        lds[t] += add;
        __syncthreads();
    }
    const unsigned long long incl = lds[t];
    total = lds[255];
    __syncthreads();
    return incl - x;
}

__device__ __forceinline__ CompactGeom item_geom(const ItemDesc& D) {
    const unsigned long long* cnt = D.counters;
    return compact_geom(cnt[CNT_PAIRS], cnt[CNT_CHUNKS], cnt[CNT_PARTIALS], D.partial_cap, D.capacity, D.slack,
                        D.chunk_shift);
}

__global__ __launch_bounds__(256) void compact_plan_kernel(const ItemDesc* __restrict__ items,
                                                           uint32_t* __restrict__ error) {
    __shared__ unsigned long long lds[256];
    const ItemDesc& D = items[blockIdx.x];
    const CompactGeom g = item_geom(D);
    const unsigned long long nd_cap = 2ull * D.partial_cap + 2ull;
    const unsigned long long nd = umin64(g.nd, nd_cap);   // g.nd <= nd_cap always (see the bounds)
    unsigned long long* Hs = D.plan;
    unsigned long long* Ds = D.plan + D.partial_cap + 1;
    const unsigned long long* pl = D.partials;

    unsigned long long run = 0, tot = 0;
    for (unsigned long long b = 0; b < g.P; b += 256) {
        const unsigned long long q = b + threadIdx.x;
        const unsigned long long len = q < g.P ? hole_len(g, pl[2 * q], pl[2 * q + 1]) : 0ull;
        const unsigned long long ex = block_exclusive_scan_u64(len, lds, tot);
        if (q < g.P) Hs[q] = run + ex;
        run += tot;
    }
    const unsigned long long TH = run;

    // fills of the data chunks: full, except the partly filled ones (each
    // chunk is on the partial list at most once)
    for (unsigned long long i = threadIdx.x; i < nd; i += 256) Ds[i] = g.C;
    __syncthreads();
    for (unsigned long long q = threadIdx.x; q < g.P; q += 256) {
        const unsigned long long c = pl[2 * q];
        if (c >= g.c0 && c - g.c0 < nd) Ds[c - g.c0] = pl[2 * q + 1];
    }
    __syncthreads();
    run = 0;
    for (unsigned long long b = 0; b < nd; b += 256) {
        const unsigned long long i = b + threadIdx.x;
        const unsigned long long len = i < nd ? data_len(g, i, Ds[i]) : 0ull;
        const unsigned long long ex = block_exclusive_scan_u64(len, lds, tot);   // every read precedes the writes
        if (i < nd) Ds[i] = run + ex;
        run += tot;
    }
    const unsigned long long TD = run;
    if (threadIdx.x == 0) {
        Hs[g.P] = TH;
        Ds[nd] = TD;
        const unsigned long long moved = umin64(TH, TD);
        D.counters[CNT_MOVED] = moved;
        D.counters[CNT_ND] = nd;
        D.counters[CNT_STORED] = g.target - (TH - moved);
        if (TH > moved || g.nd > nd_cap) atomicOr(error, (uint32_t)ERR_UNFILLED);   // never expected
    }
}

constexpr uint32_t kMoveRun = 16;   // moved elements per lane and step

// Two mappings of moved elements to lanes.  With chunks of 2^10 or more
// pairs (long holes and data runs) each wave moves a block of kWave *
// kMoveRun consecutive elements, lane l taking e0 + l, e0 + l + kWave, ...,
// so the 64 lanes of one access read and write whole cache lines (frame:
// 258 -> 95 us).  With smaller chunks a lane stepping by kWave would cross a
// hole boundary, a dependent load, almost every step; there each lane moves
// its own run of kMoveRun consecutive elements instead.  A boundary may be
// thousands of empty holes wide (300,000 eyes x 2^14 lights into 2^26 pairs,
// 4.1e5 pairs in 8,192 chunks: 33 or 700 .. 1,100 us, by the order in which the
// waves ended, with a read for each; 39 us with prefix_advance).
__global__ __launch_bounds__(256) void compact_move_kernel(const ItemDesc* __restrict__ items) {
    const ItemDesc& D = items[blockIdx.y];
    const unsigned long long moved = D.counters[CNT_MOVED];
    if (moved == 0) return;
    const CompactGeom g = item_geom(D);
    const unsigned long long nd = D.counters[CNT_ND];
    const unsigned long long* Hs = D.plan;
    const unsigned long long* Ds = D.plan + D.partial_cap + 1;
    const unsigned long long* pl = D.partials;
    uint2* out = reinterpret_cast<uint2*>(D.pairs);
    const uint2* sl = reinterpret_cast<const uint2*>(D.slack_pairs);
    const unsigned long long cap = D.capacity;
    const unsigned long long tid = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool lanes = D.chunk_shift >= 10;   // uniform over the block (one item per blockIdx.y)
    const MoveMap mm = move_map(lanes, tid, (unsigned long long)gridDim.x * blockDim.x, kMoveRun);
    for (unsigned long long e0 = mm.first; e0 < moved; e0 += mm.step) {
        // moved < both totals, so the walks below stop inside the prefixes
        unsigned long long q = prefix_rank(Hs, g.P, e0);
        unsigned long long i = prefix_rank(Ds, nd, e0);
        const unsigned long long e1 = move_run_end(mm, e0, moved);
        for (unsigned long long e = e0; e < e1; e += mm.stride) {
            q = prefix_advance(Hs, g.P, q, e);
            i = prefix_advance(Ds, nd, i, e);
            const unsigned long long dst = hole_lo(g, pl[2 * q], pl[2 * q + 1]) + (e - Hs[q]);
            const unsigned long long src = data_lo(g, i) + (e - Ds[i]);
            out[dst] = src < cap ? out[src] : sl[src - cap];
            if (D.weights) D.weights[dst] = src < cap ? D.weights[src] : D.slack_weights[src - cap];
        }
    }
}

// ---------------------------------------------------------------------------
// the allocation-free traversal: set-up and result kernels
// ---------------------------------------------------------------------------

// Writes the launch's item and task tables into the scratch header and
// clears its queue heads, counters and status words (a kernel, not a memset
// or a copy, so that the call records only kernel launches).
__global__ __launch_bounds__(256) void noalloc_setup_kernel(ItemDesc D, uint32_t n_tasks, unsigned char* base) {
    uint32_t* q = reinterpret_cast<uint32_t*>(base + kNoAllocQueues);
    for (uint32_t t = threadIdx.x; t < kQueues * kQueueStride; t += blockDim.x) q[t] = 0u;
    unsigned long long* c = reinterpret_cast<unsigned long long*>(base + kNoAllocCounters);
    for (uint32_t t = threadIdx.x; t < CNT_STRIDE; t += blockDim.x) c[t] = 0ull;
    unsigned long long* m = reinterpret_cast<unsigned long long*>(base + kNoAllocMisc);
    for (uint32_t t = threadIdx.x; t < 16u; t += blockDim.x) m[t] = 0ull;
    if (threadIdx.x == 0) {
        *reinterpret_cast<ItemDesc*>(base + kNoAllocItem) = D;
        uint32_t* tb = reinterpret_cast<uint32_t*>(base + kNoAllocTasks);
        tb[0] = 0u;
        tb[1] = n_tasks;
    }
}

// result[0] = the item's true pair count, result[1] = the status word (0 when
// the launch and its compaction completed).
__global__ void noalloc_finish_kernel(const unsigned char* base, unsigned long long* result) {
    if (threadIdx.x == 0) {
        result[0] = reinterpret_cast<const unsigned long long*>(base + kNoAllocCounters)[CNT_PAIRS];
        result[1] = reinterpret_cast<const unsigned long long*>(base + kNoAllocMisc)[1] & 0xFFFFFFFFull;
    }
}

}  // namespace hrr

// Scratch of the allocation-free traversal.  Every GPU the library runs on
// holds its own copy for the life of the process; host code reaches it only
// through the per-device address below (the array's name is not a device
// address in host code).
static __device__ __align__(256) unsigned char scratch[hrr::kNoAllocScratchBytes];

// Device address of this GPU's scratch, looked up once per device with that
// device current (called by hrr_create) and kept.
extern "C" hipError_t hrr_noalloc_scratch(int device, void** out) {
    static std::mutex mu;
    static void* addr[64] = {};
    if (device < 0 || device >= 64 || !out) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

extern "C" hipError_t hrr_launch_noalloc_setup(const hrr::ItemDesc* D, uint32_t n_tasks, void* base,
                                               hipStream_t stream) {
    hipLaunchKernelGGL(hrr::noalloc_setup_kernel, dim3(1), dim3(256), 0, stream, *D, n_tasks,
                       static_cast<unsigned char*>(base));
    return hipGetLastError();
}

extern "C" hipError_t hrr_launch_noalloc_finish(const void* base, unsigned long long* result, hipStream_t stream) {
    hipLaunchKernelGGL(hrr::noalloc_finish_kernel, dim3(1), dim3(64), 0, stream,
                       static_cast<const unsigned char*>(base), result);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launchers (called from the C++ runtime)
// ---------------------------------------------------------------------------

extern "C" hipError_t hrr_launch_rmq(const uint32_t* a, const uint32_t* b, const uint32_t* r, uint64_t n,
                                     uint32_t method, uint32_t* k, uint32_t* v, unsigned long long* n_bad,
                                     int n_cu, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int vec = ((((uintptr_t)a) | ((uintptr_t)b) | ((uintptr_t)r) | ((uintptr_t)k) | ((uintptr_t)v)) & 15u) == 0;
    const uint64_t work = vec ? (n + 3) / 4 : n;
    // kRmqGroups 4-query groups per thread and a grid far larger than the
    // resident capacity keep the most loads in flight (2^28 queries with
    // ordinary loads: 1.26 ms with 16 blocks per CU and a grid-stride loop,
    // 1.02 ms with one group per thread, 0.98 ms with two; with non-temporal
    // loads one group is best).  The loop still covers grids above the cap.
    const uint64_t per_block = vec ? 256ull * hrr::kRmqGroups : 256ull;
    uint64_t blocks = (work + per_block - 1) / per_block;
    const uint64_t max_blocks = 1ull << 30;
    (void)n_cu;
    if (blocks > max_blocks) blocks = max_blocks;
    if (blocks < 1) blocks = 1;
    if (method == 1)
        hipLaunchKernelGGL(hrr::rmq_kernel<1>, dim3((uint32_t)blocks), dim3(256), 0, stream, a, b, r, n, k, v, n_bad, vec);
    else if (method == 2)
        hipLaunchKernelGGL(hrr::rmq_kernel<2>, dim3((uint32_t)blocks), dim3(256), 0, stream, a, b, r, n, k, v, n_bad, vec);
    else if (method == 3)
        hipLaunchKernelGGL(hrr::rmq_kernel<3>, dim3((uint32_t)blocks), dim3(256), 0, stream, a, b, r, n, k, v, n_bad, vec);
    else if (method == 4)
        hipLaunchKernelGGL(hrr::rmq_kernel<4>, dim3((uint32_t)blocks), dim3(256), 0, stream, a, b, r, n, k, v, n_bad, vec);
    else
        hipLaunchKernelGGL(hrr::rmq_kernel<0>, dim3((uint32_t)blocks), dim3(256), 0, stream, a, b, r, n, k, v, n_bad, vec);
    return hipGetLastError();
}

// Compaction of a launch's items (see compact_plan_kernel): n_items <= 65535.
extern "C" hipError_t hrr_launch_compact(const hrr::ItemDesc* items, uint32_t n_items, uint32_t* error,
                                         hipStream_t stream) {
    if (n_items == 0) return hipSuccess;
    if (n_items > 65535u) return hipErrorInvalidValue;
    hipLaunchKernelGGL(hrr::compact_plan_kernel, dim3(n_items), dim3(256), 0, stream, items, error);
    // about 8192 blocks in all, at least 16 and at most 4096 per item
    uint32_t per_item = 8192u / n_items;
    per_item = per_item < 16u ? 16u : (per_item > 4096u ? 4096u : per_item);
    hipLaunchKernelGGL(hrr::compact_move_kernel, dim3(per_item, n_items), dim3(256), 0, stream, items);
    return hipGetLastError();
}

namespace {

template <int EPW, int METHOD, bool STATS, bool W>
hipError_t launch_trav(const hrr::TravArgs& A, uint32_t blocks, size_t lds, hipStream_t stream) {
    auto kern = hrr::traverse_kernel<EPW, METHOD, STATS, W>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(hrr::kWave * hrr::kWavesPerBlock), lds, stream, A);
    return hipGetLastError();
}

template <int EPW, int METHOD, bool STATS>
hipError_t pick_w(const hrr::TravArgs& A, bool w, uint32_t blocks, size_t lds, hipStream_t s) {
    return w ? launch_trav<EPW, METHOD, STATS, true>(A, blocks, lds, s)
             : launch_trav<EPW, METHOD, STATS, false>(A, blocks, lds, s);
}

template <int EPW, int METHOD>
hipError_t pick_stats(const hrr::TravArgs& A, bool st, bool w, uint32_t blocks, size_t lds, hipStream_t s) {
    return st ? pick_w<EPW, METHOD, true>(A, w, blocks, lds, s) : pick_w<EPW, METHOD, false>(A, w, blocks, lds, s);
}

template <int EPW>
hipError_t pick_method(const hrr::TravArgs& A, uint32_t method, bool st, bool w, uint32_t blocks, size_t lds,
                       hipStream_t s) {
    if (method == 1) return pick_stats<EPW, 1>(A, st, w, blocks, lds, s);
    if (method == 2) return pick_stats<EPW, 2>(A, st, w, blocks, lds, s);
    if (method == 3) return pick_stats<EPW, 3>(A, st, w, blocks, lds, s);
    if (method == 4) return pick_stats<EPW, 4>(A, st, w, blocks, lds, s);
    if (method == 5) return pick_stats<EPW, 5>(A, st, w, blocks, lds, s);
    return pick_stats<EPW, 0>(A, st, w, blocks, lds, s);
}

}  // namespace

// LDS bytes of one wave for a given stack size.
extern "C" size_t hrr_trav_lds_per_wave(uint32_t stack_cap, uint32_t eyes_per_wave) {
    return (size_t)stack_cap * sizeof(uint2) + (eyes_per_wave > 1 ? hrr::kEyeTableBytes : hrr::kXposeBytes);
}

// Dynamic LDS bytes of one block.
extern "C" size_t hrr_trav_lds_per_block(uint32_t n_items, size_t lds_per_wave) {
    return ((size_t)n_items + 1u) * sizeof(uint32_t) / 16u * 16u + 16u + lds_per_wave * hrr::kWavesPerBlock;
}

extern "C" hipError_t hrr_launch_traverse(const hrr::TravArgs* A, uint32_t eyes_per_wave, uint32_t method,
                                          int stats, int with_weights, uint32_t blocks, hipStream_t stream) {
    const size_t lds = hrr_trav_lds_per_block(A->n_items, A->lds_per_wave);
    switch (eyes_per_wave) {
        case 1: return pick_method<1>(*A, method, stats, with_weights, blocks, lds, stream);
        case 2: return pick_method<2>(*A, method, stats, with_weights, blocks, lds, stream);
        case 4: return pick_method<4>(*A, method, stats, with_weights, blocks, lds, stream);
        case 8: return pick_method<8>(*A, method, stats, with_weights, blocks, lds, stream);
        default: return hipErrorInvalidValue;
    }
}

// Resident blocks per CU for a launch shape (for sizing the persistent grid).
extern "C" hipError_t hrr_traverse_occupancy(uint32_t eyes_per_wave, uint32_t method, int stats, int with_weights,
                                             size_t lds_per_block, int* blocks_per_cu) {
    const void* f = nullptr;
#define HRR_PICK(E, M, S, W) \
    if (eyes_per_wave == E && method == M && (stats != 0) == S && (with_weights != 0) == W) \
        f = (const void*)hrr::traverse_kernel<E, M, S, W>;
#define HRR_PICK_SW(E, M) HRR_PICK(E, M, false, false) HRR_PICK(E, M, false, true) HRR_PICK(E, M, true, false) HRR_PICK(E, M, true, true)
#define HRR_PICK_M(E) \
    HRR_PICK_SW(E, 0) HRR_PICK_SW(E, 1) HRR_PICK_SW(E, 2) HRR_PICK_SW(E, 3) HRR_PICK_SW(E, 4) HRR_PICK_SW(E, 5)
    HRR_PICK_M(1) HRR_PICK_M(2) HRR_PICK_M(4) HRR_PICK_M(8)
#undef HRR_PICK_M
#undef HRR_PICK_SW
#undef HRR_PICK
    if (!f) return hipErrorInvalidValue;
    if (lds_per_block > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_per_block);
        if (e != hipSuccess) return e;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, f, hrr::kWave * hrr::kWavesPerBlock,
                                                        lds_per_block);
}

// Dynamic LDS bytes of one block of the block walk.
extern "C" size_t hrr_cull_lds_per_block(uint32_t n_items, int with_weights, int dense) {
    return hrr::kWavesPerBlock * hrr::cull_wave_bytes(with_weights != 0, dense != 0) +
           ((size_t)n_items + 1u) * sizeof(uint32_t);
}

namespace {
typedef void (*CullKernel)(hrr::TravArgs);
CullKernel pick_cull(int with_weights, int dense) {
    if (with_weights) return dense ? hrr::cull_kernel<true, true> : hrr::cull_kernel<true, false>;
    return dense ? hrr::cull_kernel<false, true> : hrr::cull_kernel<false, false>;
}
}  // namespace

// The block walk (see cull_kernel) of a launch's items.
extern "C" hipError_t hrr_launch_cull(const hrr::TravArgs* A, int with_weights, int dense, uint32_t blocks,
                                      hipStream_t stream) {
    hipLaunchKernelGGL(pick_cull(with_weights, dense), dim3(blocks), dim3(hrr::kWave * hrr::kWavesPerBlock),
                       hrr_cull_lds_per_block(A->n_items, with_weights, dense), stream, *A);
    return hipGetLastError();
}

// Resident blocks per CU of the block walk.
extern "C" hipError_t hrr_cull_occupancy(int with_weights, int dense, uint32_t n_items, int* blocks_per_cu) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void*)pick_cull(with_weights, dense),
                                                        hrr::kWave * hrr::kWavesPerBlock,
                                                        hrr_cull_lds_per_block(n_items, with_weights, dense));
}

// The block tree of n_lights >= 1 lights (float4 in sequence order): blocks
// holds block_tree_slots(block_tree_log(n_lights)) boxes.
extern "C" hipError_t hrr_launch_blocks(const float* lights, uint32_t n_lights, float* blocks, hipStream_t stream) {
    const uint32_t log = hrr::block_tree_log(n_lights);
    uint32_t level = (log - hrr::block_leaf_log(log)) / 2u;
    float4* out = reinterpret_cast<float4*>(blocks);
    hipLaunchKernelGGL(hrr::block_leaf_kernel, dim3(((1u << (2u * level)) + 255u) / 256u), dim3(256), 0, stream,
                       reinterpret_cast<const float4*>(lights), n_lights, log, out,
                       reinterpret_cast<float4*>(blocks + hrr::block_lights_at(n_lights)));
    for (; level > 4u; level -= 4u)
        hipLaunchKernelGGL(hrr::block_up_kernel, dim3(((1u << (2u * (level - 4u))) + 255u) / 256u), dim3(256), 0, stream,
                           level - 4u, out);
    return hipGetLastError();
}

// The top of a hierarchy with records (see frontier_kernel): out holds
// kFrontierWords words; blocks is the lights' block tree.
extern "C" hipError_t hrr_launch_frontier(const hrr::Node* nodes, uint32_t n_lights, uint32_t leaf_size,
                                          const float* blocks, float* out, hipStream_t stream) {
    hipLaunchKernelGGL(hrr::frontier_kernel, dim3(2), dim3(64), 0, stream, nodes, n_lights, leaf_size,
                       reinterpret_cast<const float4*>(blocks), out);
    return hipGetLastError();
}

// Processing order of the virtual eyes of a launch (see order_keys_kernel).
// hist must hold (n_items << (3 bits + rbits)) + 1024 counters (the last 1024
// are the scan's chunk sums); keys and order `total` words; tile is the
// context's 64x64 tile, whose values share tile_tz trailing zeros (rbits = 0
// leaves the shift out of the key).
extern "C" hipError_t hrr_launch_order(const hrr::OrderItem* items, const uint32_t* vbegin, uint32_t n_items,
                                       uint32_t total, uint32_t bits, uint32_t rbits, const uint32_t* tile,
                                       uint32_t tile_tz, uint32_t* keys, uint32_t* hist, uint32_t* order, int n_cu,
                                       hipStream_t stream) {
    if (total == 0) return hipSuccess;
    if (rbits > 31u || (rbits && tile_tz > 31u)) return hipErrorInvalidValue;
    const uint32_t key_bits = 3u * bits + rbits;
    const uint32_t n_buckets = n_items << key_bits;
    if (hrr::scan::chunk_count(n_buckets) > 1024u) return hipErrorInvalidValue;
    hipError_t e = hipMemsetAsync(hist, 0, (size_t)n_buckets * sizeof(uint32_t), stream);
    if (e != hipSuccess) return e;
    uint32_t blocks = (total + 255u) / 256u;
    const uint32_t max_blocks = (uint32_t)(n_cu > 0 ? n_cu : 256) * 8u;
    if (blocks > max_blocks) blocks = max_blocks;
    hipLaunchKernelGGL(hrr::order_keys_kernel, dim3(blocks), dim3(256), 0, stream, items, vbegin, n_items, total, bits,
                       rbits, tile, tile_tz, keys, hist);
    if ((e = hrr::scan::exclusive_sum(hist, hist, n_buckets, hist + n_buckets, stream)) != hipSuccess) return e;
    hipLaunchKernelGGL(hrr::order_scatter_kernel, dim3(blocks), dim3(256), 0, stream, keys, vbegin, total, key_bits,
                       hist, order);
    return hipGetLastError();
}
