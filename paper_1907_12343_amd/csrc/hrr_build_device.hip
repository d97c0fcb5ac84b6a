// hrr_build_device.hip -- the light hierarchy built on the GPU, record for
// record identical to the host builder (hrr_build.cpp): same Morton codes,
// same (code, original index) order, same split rule (radix split with the
// midpoint for equal codes, or the power-of-two split), same exact fp32 boxes
// and the same record numbering (sibling pairs in preorder of their owners).
//
// Section 1 of the paper only needs the lights sorted by a spatial hierarchy
// with every node a contiguous index range; building it on the device lets a
// renderer rebuild per-frame light caches without a host round trip.
//
// Steps (all stream-ordered; the host waits twice, for the record count and
// for the end):
//   1. codes   : 63-bit Morton code per light (21-bit cells, x highest)
//   2. sort    : stable LSD radix sort of (code, index) pairs, 8-bit digits
//   3. gather  : lights and original indices in sequence order, then the
//                block tree of the lights (block_leaf_kernel, hrr_kernels.hip)
//   4. nodes   : one thread per index c in (0, n): a full binary tree over n
//                lights has one node per split position, and both split rules
//                give that node's range [a, b) and its parent from c alone
//                (see node_of)
//   5. ranks   : record numbers.  Owners (nodes with an internal child) before
//                a node in preorder are those that start at a smaller index,
//                an exclusive scan, and the ancestors that start at the same
//                one, its chain of left-child steps up
//   6. records : the 64-byte records, children's boxes from the lights of
//                small children and from the block tree of large ones
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdint.h>

#include "hrr_devbuild.hpp"
#include "hrr_scan.hpp"
#include "hrr_types.hpp"

namespace hrr {
namespace devbuild {

// ---- Morton code, written out as in the host builder --------------------

__device__ __forceinline__ uint64_t spread_bits3(uint32_t v) {
    uint64_t x = v & 0x1FFFFFu;
    x = (x | (x << 32)) & 0x001F00000000FFFFull;
    x = (x | (x << 16)) & 0x001F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ __forceinline__ uint32_t cell21(float x, float lo, float hi) {
    float u = (x - lo) / (hi - lo);
    if (!(u > 0.0f)) u = 0.0f;
    if (u > 1.0f) u = 1.0f;
    const uint32_t q = (uint32_t)(u * 2097152.0f);
    return q < 2097151u ? q : 2097151u;
}

__global__ void codes_kernel(const float* __restrict__ xyz, uint32_t n, QBox qb, uint64_t* __restrict__ code,
                             uint32_t* __restrict__ idx, uint32_t* __restrict__ bad) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = xyz[3 * (size_t)i], y = xyz[3 * (size_t)i + 1], z = xyz[3 * (size_t)i + 2];
    if (!isfinite(x) || !isfinite(y) || !isfinite(z)) atomicOr(bad, 1u);
    code[i] = (spread_bits3(cell21(x, qb.lo[0], qb.hi[0])) << 2) | (spread_bits3(cell21(y, qb.lo[1], qb.hi[1])) << 1) |
              spread_bits3(cell21(z, qb.lo[2], qb.hi[2]));
    idx[i] = i;
}

__global__ void gather_kernel(const float* __restrict__ xyz, const uint32_t* __restrict__ order, uint32_t n,
                              float4* __restrict__ lights, uint32_t* __restrict__ perm) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t j = order[i];
    lights[i] = make_float4(xyz[3 * (size_t)j], xyz[3 * (size_t)j + 1], xyz[3 * (size_t)j + 2], 0.0f);
    perm[i] = j;
}

// ---- nodes by split position ----------------------------------------------
//
// Radix split: the node that is cut between c - 1 and c at code bit h holds
// exactly the lights that share the code bits above h with light c, a range
// around c found by galloping outwards (most nodes are small).  Lights of one
// code form a run [p, q), whose subtree is cut at midpoints: there the node is
// found by descending from [p, q).  The parent of a node [a, b) is cut at a or
// at b, at the position whose codes differ in the lower bit (the two never
// tie: between two cuts at one bit lies one at a higher bit).
// Power-of-two split: with 2^t the lowest set bit of c the node is
// [c - 2^t, min(c + 2^t, n)), and its parent's cut follows from the next bit.

// Parent of a node: its split position << 1 | 1 for a right child.
constexpr uint32_t kNoParent = 0xFFFFFFFFu;

struct NodeAt {
    uint32_t a, b, parent;
};

// bit in which the codes on both sides of boundary x differ (-1: equal codes)
__device__ __forceinline__ int cut_bit(const uint64_t* __restrict__ code, uint32_t n, uint32_t x) {
    if (x == 0u || x == n) return 64;
    const uint64_t d = code[x - 1u] ^ code[x];
    return d ? 63 - __clzll((long long)d) : -1;
}

// The largest range around c (c - 1 and c inside) whose codes >> shift equal
// code[c] >> shift.
__device__ __forceinline__ void same_prefix_range(const uint64_t* __restrict__ code, uint32_t n, uint32_t c,
                                                  uint32_t shift, uint32_t* a, uint32_t* b) {
    const uint64_t prefix = code[c] >> shift;
    uint32_t lo = c - 1u, hi = c, step = 1;
    while (lo >= step && (code[lo - step] >> shift) == prefix) {
        lo -= step;
        step <<= 1;
    }
    for (; step; step >>= 1)
        if (lo >= step && (code[lo - step] >> shift) == prefix) lo -= step;
    step = 1;
    while (n - hi > step && (code[hi + step] >> shift) == prefix) {
        hi += step;
        step <<= 1;
    }
    for (; step; step >>= 1)
        if (n - hi > step && (code[hi + step] >> shift) == prefix) hi += step;
    *a = lo;
    *b = hi + 1u;
}

__device__ __forceinline__ NodeAt node_of(const uint64_t* __restrict__ code, uint32_t n, uint32_t c, uint32_t pow2) {
    NodeAt r;
    if (pow2) {
        const uint32_t t = 1u << (uint32_t)__builtin_ctz(c);
        r.a = c - t;
        r.b = n - c > t ? c + t : n;
        if (r.a == 0u && r.b == n) r.parent = kNoParent;
        else if (r.b < n && !(r.a & (2u * t))) r.parent = r.b << 1;
        else r.parent = (r.a << 1) | 1u;
        return r;
    }
    const int h = cut_bit(code, n, c);
    same_prefix_range(code, n, c, (uint32_t)(h + 1), &r.a, &r.b);
    const int l = cut_bit(code, n, r.a), u = cut_bit(code, n, r.b);
    r.parent = r.a == 0u && r.b == n ? kNoParent : (l < u ? (r.a << 1) | 1u : r.b << 1);
    if (h < 0) {
        for (;;) {
            const uint32_t mid = r.a + (r.b - r.a) / 2u;
            if (mid == c) break;
            if (c < mid) {
                r.b = mid;
                r.parent = mid << 1;
            } else {
                r.a = mid;
                r.parent = (mid << 1) | 1u;
            }
        }
    }
    return r;
}

// Tables by split position c: range (b = 0: not an internal node), parent,
// record number of the children's pair; owners by first index.
__global__ __launch_bounds__(256) void nodes_kernel(const uint64_t* __restrict__ code, uint32_t n, uint32_t leaf,
                                                    uint32_t pow2, uint2* __restrict__ range,
                                                    uint32_t* __restrict__ parent, uint32_t* __restrict__ owners) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x + 1u;
    if (c >= n) return;
    const NodeAt r = node_of(code, n, c, pow2);
    const bool internal = r.b - r.a > leaf;
    range[c] = internal ? make_uint2(r.a, r.b) : make_uint2(0u, 0u);
    parent[c] = r.parent;
    if (internal && (c - r.a > leaf || r.b - c > leaf)) atomicAdd(owners + r.a, 1u);
}

// before: the exclusive scan of the owners by first index (n + 1 entries).
// out[0] = all owners, out[1] = the deepest node's depth (zero before).
__global__ __launch_bounds__(256) void ranks_kernel(const uint2* __restrict__ range, const uint32_t* __restrict__ parent,
                                                    const uint32_t* __restrict__ before, uint32_t n, uint32_t leaf,
                                                    uint32_t* __restrict__ first, uint32_t* __restrict__ out) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x + 1u;
    if (c == 1u) out[0] = before[n];
    uint32_t depth = 0;
    if (c < n && range[c].y != 0u) {
        const uint2 r = range[c];
        const bool owner = c - r.x > leaf || r.y - c > leaf;
        uint32_t p = parent[c], chain = 0;
        for (; p != kNoParent && !(p & 1u); ++chain) p = parent[p >> 1];   // every one of them is an owner
        first[c] = owner ? 2u * (1u + before[r.x] + chain) : 0xFFFFFFFFu;
        if (!owner)
            for (depth = chain; p != kNoParent; ++depth) p = parent[p >> 1];
    }
    for (int o = 32; o > 0; o >>= 1) depth = max(depth, (uint32_t)__shfl_xor((int)depth, o));
    // few waves raise the maximum: look before adding to the one address
    if ((threadIdx.x & 63u) == 0u && depth > __hip_atomic_load(out + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(out + 1, depth);
}

__device__ __forceinline__ void widen(float* lo, float* hi, const float4& l, const float4& h) {
    lo[0] = min_first(lo[0], l.x); hi[0] = max_first(hi[0], h.x);
    lo[1] = min_first(lo[1], l.y); hi[1] = max_first(hi[1], h.y);
    lo[2] = min_first(lo[2], l.z); hi[2] = max_first(hi[2], h.z);
}

// Box of the lights [a, b), which the host builder computes light by light and
// child by child: the first light (in sequence order) that attains each bound
// gives it, so lights and whole blocks are taken in order here.
__device__ __forceinline__ void range_box(const float4* __restrict__ lights, const float4* __restrict__ blocks,
                                          uint32_t block_log, uint32_t a, uint32_t b, float* lo, float* hi) {
    const uint32_t leaf_log = block_leaf_log(block_log), small = 1u << leaf_log;
    const float4 p = lights[a];
    lo[0] = hi[0] = p.x;
    lo[1] = hi[1] = p.y;
    lo[2] = hi[2] = p.z;
    for (uint32_t i = b - a < small ? a + 1u : a; i < b;) {
        if ((i & (small - 1u)) == 0u && b - i >= small) {
            uint32_t v = leaf_log;
            while (v + 2u < block_log && (i & ((4u << v) - 1u)) == 0u && (b - i) >> v >= 4u) v += 2u;
            const uint32_t id = (1u << (block_log - v)) + (i >> v);
            widen(lo, hi, blocks[2u * id], blocks[2u * id + 1u]);
            i += 1u << v;
        } else {
            const float4 q = lights[i];
            widen(lo, hi, q, q);
            ++i;
        }
    }
}

// Bound by the scattered 64-byte stores and the lights' loads: 39 us for 2^20
// lights (67 MB of records); the nodes and ranks before it 20 and 36 .. 73 us,
// the sort 210 us.  A build of 2^20 lights takes 0.49 ms against 3.9 ms with one
// launch and one host wait per tree level.
__global__ __launch_bounds__(256) void records_kernel(const uint2* __restrict__ range, const uint32_t* __restrict__ parent,
                                                      const uint32_t* __restrict__ first,
                                                      const float4* __restrict__ lights,
                                                      const float4* __restrict__ blocks, uint32_t block_log, uint32_t n,
                                                      Node* __restrict__ nodes) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x + 1u;
    if (c >= n) return;
    const uint2 r = range[c];
    if (r.y == 0u) return;
    const uint32_t p = parent[c];
    Node nd;
    range_box(lights, blocks, block_log, r.x, c, nd.lo_l, nd.hi_l);
    range_box(lights, blocks, block_log, c, r.y, nd.lo_r, nd.hi_r);
    nd.a = r.x;
    nd.c = c;
    nd.b = r.y;
    nd.first = first[c];
    nodes[p == kNoParent ? 0u : first[p >> 1] + (p & 1u)] = nd;
}

// ---- stable LSD radix sort of (code, index) pairs ----------------------
//
// Eight passes of 8-bit digits cover the 63 code bits, least significant
// digit first.  One pass counts the digits of every tile of 256 ROUNDS keys
// and scatters each tile's keys stably.  A wave owns a run of 64 ROUNDS
// consecutive keys of its tile and takes them 64 at a time: a key's rank in the
// run is the number of its digit's keys in earlier rounds (an LDS count that
// only this wave touches) plus those in earlier lanes (found with eight
// ballots, one per digit bit).  The keys stay in registers while the waves'
// counts become first positions, so a tile needs two barriers however many
// rounds it has (2^20 keys: 20 us a scatter with two barriers a round).  Keys
// of one digit leave in index order, which makes every pass stable and the
// result ordered by (code, original index).

constexpr uint32_t kSortThreads = 256;
constexpr uint32_t kSortWaves = kSortThreads / 64;
constexpr uint32_t kSortDigits = 256;
constexpr uint32_t kSortPasses = 8;

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Lanes of the wave (among `valid`) whose digit equals this lane's.
__device__ __forceinline__ uint64_t same_digit_lanes(uint32_t d, uint64_t valid) {
    uint64_t peers = valid;
#pragma unroll
    for (uint32_t bit = 0; bit < 8u; ++bit) {
        const bool set = (d >> bit) & 1u;
        const uint64_t m = __builtin_amdgcn_ballot_w64(set);
        peers &= set ? m : ~m;
    }
    return peers;
}

// counts: tile-major with FUSED (see sort_pass), digit-major else.
template <uint32_t ROUNDS, bool FUSED>
__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(const uint64_t* __restrict__ key, uint32_t n,
                                                                  uint32_t shift, uint32_t n_tiles,
                                                                  uint32_t* __restrict__ counts) {
    __shared__ uint32_t hist[kSortWaves][kSortDigits];   // a wave's own counts
    const uint32_t t = threadIdx.x, w = t >> 6;
    for (uint32_t q = 0; q < kSortWaves; ++q) hist[q][t] = 0u;
    __syncthreads();
    const uint32_t base = blockIdx.x * kSortThreads * ROUNDS;
#pragma unroll
    for (uint32_t r = 0; r < ROUNDS; ++r) {
        const uint32_t i = base + r * kSortThreads + t;
        if (i < n) atomicAdd(&hist[w][(uint32_t)(key[i] >> shift) & (kSortDigits - 1u)], 1u);
    }
    __syncthreads();
    uint32_t sum = 0;
    for (uint32_t q = 0; q < kSortWaves; ++q) sum += hist[q][t];
    counts[FUSED ? (size_t)blockIdx.x * kSortDigits + t : (size_t)t * n_tiles + blockIdx.x] = sum;
}

// One block per digit: its counts (digit-major, n_tiles of them) become their
// exclusive prefix sums in tile order, totals[d] their sum.
constexpr uint32_t kRowCounts = 8;   // a thread's counts per step
__global__ __launch_bounds__(kSortThreads) void sort_rows_kernel(uint32_t* __restrict__ counts, uint32_t n_tiles,
                                                                 uint32_t* __restrict__ totals) {
    __shared__ uint32_t lds[4];
    uint32_t* const row = counts + (size_t)blockIdx.x * n_tiles;
    uint32_t carry = 0;
    for (uint32_t b = threadIdx.x * kRowCounts; b - threadIdx.x * kRowCounts < n_tiles; b += kSortThreads * kRowCounts) {
        uint32_t x[kRowCounts], sum = 0, total;
#pragma unroll
        for (uint32_t q = 0; q < kRowCounts; ++q) {
            x[q] = b + q < n_tiles ? row[b + q] : 0u;
            sum += x[q];
        }
        uint32_t run = carry + scan::block_inclusive_256(sum, lds, &total) - sum;
#pragma unroll
        for (uint32_t q = 0; q < kRowCounts; ++q) {
            if (b + q < n_tiles) row[b + q] = run;
            run += x[q];
        }
        carry += total;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// first, totals: the tiles' counts with FUSED, else what sort_rows_kernel wrote.
template <uint32_t ROUNDS, bool FUSED>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(const uint64_t* __restrict__ kin,
                                                                    const uint32_t* __restrict__ vin, uint32_t n,
                                                                    uint32_t shift, uint32_t n_tiles,
                                                                    const uint32_t* __restrict__ first,
                                                                    const uint32_t* __restrict__ totals,
                                                                    uint64_t* __restrict__ kout,
                                                                    uint32_t* __restrict__ vout) {
    // pos[w][d]: keys of digit d in wave w's run, then their first position
    __shared__ uint32_t pos[kSortWaves][kSortDigits];
    const uint32_t t = threadIdx.x, w = t >> 6, lane = t & 63u;
    for (uint32_t q = 0; q < kSortWaves; ++q) pos[q][t] = 0u;
    __syncthreads();
    const uint32_t base = (blockIdx.x * kSortWaves + w) * 64u * ROUNDS;
    uint64_t k[ROUNDS];
    uint32_t v[ROUNDS], rank[ROUNDS];
#pragma unroll
    for (uint32_t r = 0; r < ROUNDS; ++r) {
        const uint32_t i = base + r * 64u + lane;
        k[r] = i < n ? kin[i] : 0ull;
        v[r] = i < n ? vin[i] : 0u;
    }
    // this tile's first position of digit t (the loads overlap the ranking)
    uint32_t start;
    if (FUSED) {
        // the keys of smaller digits, and those of digit t in earlier tiles
        __shared__ uint32_t lds[4];
        uint32_t all = 0, before = 0, total;
#pragma unroll 8
        for (uint32_t b = 0; b < n_tiles; ++b) {
            const uint32_t x = first[(size_t)b * kSortDigits + t];
            all += x;
            before += b < blockIdx.x ? x : 0u;
        }
        start = scan::block_inclusive_256(all, lds, &total) - all + before;
    } else {
        __shared__ uint32_t lds[4];
        uint32_t total;
        const uint32_t all = totals[t], before = first[(size_t)t * n_tiles + blockIdx.x];
        start = scan::block_inclusive_256(all, lds, &total) - all + before;
    }
#pragma unroll
    for (uint32_t r = 0; r < ROUNDS; ++r) {
        const bool ok = base + r * 64u + lane < n;
        const uint32_t d = (uint32_t)(k[r] >> shift) & (kSortDigits - 1u);
        const uint64_t peers = same_digit_lanes(d, __builtin_amdgcn_ballot_w64(ok));
        const uint32_t below = lanes_below(peers);
        const uint32_t seen = pos[w][d];
        rank[r] = seen + below;
        // every lane has read its digit's count (one wave runs in lock step,
        // its LDS accesses in order) before the first lane of each digit adds
        __builtin_amdgcn_wave_barrier();
        if (ok && below == 0u) pos[w][d] = seen + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (uint32_t q = 0; q < kSortWaves; ++q) {
        const uint32_t c = pos[q][t];
        pos[q][t] = start;
        start += c;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < ROUNDS; ++r) {
        if (base + r * 64u + lane < n) {
            const uint32_t at = pos[w][(uint32_t)(k[r] >> shift) & (kSortDigits - 1u)] + rank[r];
            kout[at] = k[r];
            vout[at] = v[r];
        }
    }
}

}  // namespace devbuild
}  // namespace hrr

using namespace hrr;
using namespace hrr::devbuild;

namespace {

constexpr uint32_t kThreads = 256;

uint32_t blocks_for(uint32_t n) { return (n + kThreads - 1) / kThreads; }

}  // namespace

// Scratch sizes and steps are driven from the host file (hrr_api.cpp) through
// these entry points; every one is asynchronous on `stream`.
extern "C" hipError_t hrr_dev_codes(const float* xyz, uint32_t n, const float* qbox, uint64_t* code, uint32_t* idx,
                                    uint32_t* bad, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    QBox qb;
    for (int k = 0; k < 3; ++k) {
        qb.lo[k] = qbox[k];
        qb.hi[k] = qbox[3 + k];
    }
    codes_kernel<<<blocks_for(n), kThreads, 0, stream>>>(xyz, n, qb, code, idx, bad);
    return hipGetLastError();
}

size_t align256(size_t b) { return (b + 255u) & ~(size_t)255u; }

// Rounds of 256 keys per tile of the sort: 8 for large inputs, fewer where that
// would leave CUs without a tile.  us a build at 2 / 4 / 8 / 16 rounds: 20,011
// lights 188 / 199 / 214 / 263, 2^17 291 / 254 / 252 / 287, 2^18 415 / 330 /
// 303 / 329, 2^20 607 / 553 / 543 / 573.
uint32_t sort_rounds(uint32_t n) { return n >= (1u << 18) ? 8u : n >= (1u << 16) ? 4u : 2u; }

// FUSED: up to kSortFused tiles every scatter block adds up the tile counts it
// needs itself (tile-major counts, 1 KB per tile out of L2) instead of launches
// between the two that scan them (three: 12 us of a pass of 20 at 20,011 keys);
// beyond, that reading grows with the square of the tiles.  There one launch
// scans each digit's counts, and the scatter blocks scan the 256 totals (2^20
// keys: 490 us a build against 560 with a three-launch scan of all counts).
// us a build, fused / with the scan: 40 tiles 186 / 195, 64 225 / 222, 128 (2^17
// keys) 252 / 236, 128 (2^18) 308 / 291.
constexpr uint32_t kSortFused = 48;

template <uint32_t ROUNDS>
hipError_t sort_pass(const uint64_t* ks, const uint32_t* vs, uint32_t n, uint32_t shift, uint32_t n_tiles,
                     uint32_t* counts, uint32_t* totals, uint64_t* kd, uint32_t* vd, hipStream_t stream) {
    if (n_tiles <= kSortFused) {
        sort_count_kernel<ROUNDS, true><<<n_tiles, kSortThreads, 0, stream>>>(ks, n, shift, n_tiles, counts);
        sort_scatter_kernel<ROUNDS, true><<<n_tiles, kSortThreads, 0, stream>>>(ks, vs, n, shift, n_tiles, counts, totals,
                                                                               kd, vd);
        return hipGetLastError();
    }
    sort_count_kernel<ROUNDS, false><<<n_tiles, kSortThreads, 0, stream>>>(ks, n, shift, n_tiles, counts);
    sort_rows_kernel<<<kSortDigits, kSortThreads, 0, stream>>>(counts, n_tiles, totals);
    sort_scatter_kernel<ROUNDS, false><<<n_tiles, kSortThreads, 0, stream>>>(ks, vs, n, shift, n_tiles, counts, totals,
                                                                            kd, vd);
    return hipGetLastError();
}

// Stable radix sort of (code, index) by code (63 low bits); temp == nullptr
// queries temp_bytes.  Scratch: a second key and index buffer (the passes
// alternate between it and the outputs, the last pass landing in the
// outputs), the per-tile digit counts and the digits' totals.
extern "C" hipError_t hrr_dev_sort(void* temp, size_t* temp_bytes, const uint64_t* code_in, uint64_t* code_out,
                                   const uint32_t* idx_in, uint32_t* idx_out, uint32_t n, hipStream_t stream) {
    static_assert(kSortPasses % 2 == 0, "the last pass must write the outputs");
    if (!temp_bytes) return hipErrorInvalidValue;
    const uint32_t rounds = sort_rounds(n), tile = kSortThreads * rounds;
    const uint32_t n_tiles = (n + tile - 1u) / tile;
    const uint32_t n_counts = n_tiles * kSortDigits;
    const size_t b_keys = align256((size_t)n * 8u), b_idx = align256((size_t)n * 4u);
    const size_t b_counts = align256((size_t)n_counts * 4u), b_totals = kSortDigits * 4u;
    const size_t need = std::max<size_t>(b_keys + b_idx + b_counts + b_totals, 256u);
    if (!temp) {
        *temp_bytes = need;
        return hipSuccess;
    }
    if (*temp_bytes < need) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    unsigned char* tp = static_cast<unsigned char*>(temp);
    uint64_t* k_tmp = reinterpret_cast<uint64_t*>(tp);
    uint32_t* v_tmp = reinterpret_cast<uint32_t*>(tp + b_keys);
    uint32_t* counts = reinterpret_cast<uint32_t*>(tp + b_keys + b_idx);
    uint32_t* totals = reinterpret_cast<uint32_t*>(tp + b_keys + b_idx + b_counts);
    const uint64_t* ks = code_in;
    const uint32_t* vs = idx_in;
    for (uint32_t pass = 0; pass < kSortPasses; ++pass) {
        uint64_t* kd = (pass & 1u) ? code_out : k_tmp;
        uint32_t* vd = (pass & 1u) ? idx_out : v_tmp;
        const uint32_t shift = 8u * pass;
        const hipError_t e = rounds == 4u ? sort_pass<4>(ks, vs, n, shift, n_tiles, counts, totals, kd, vd, stream)
                             : rounds == 8u ? sort_pass<8>(ks, vs, n, shift, n_tiles, counts, totals, kd, vd, stream)
                                          : sort_pass<2>(ks, vs, n, shift, n_tiles, counts, totals, kd, vd, stream);
        if (e != hipSuccess) return e;
        ks = kd;
        vs = vd;
    }
    return hipSuccess;
}

extern "C" hipError_t hrr_dev_gather(const float* xyz, const uint32_t* order, uint32_t n, float* lights,
                                     uint32_t* perm, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    gather_kernel<<<blocks_for(n), kThreads, 0, stream>>>(xyz, order, n, reinterpret_cast<float4*>(lights), perm);
    return hipGetLastError();
}

// Words of scratch behind the node tables (see hrr_dev_nodes), n >= 2.
extern "C" size_t hrr_dev_nodes_words(uint32_t n) {
    // range (2), parent, first: n each; owners n + 1; chunk sums of the scan
    return 5 * (size_t)n + 1 + scan::chunk_count(n + 1u) + 8;
}

namespace {
struct NodeTables {
    uint2* range;
    uint32_t *parent, *first, *owners, *sums;
    NodeTables(uint32_t* words, uint32_t n)
        : range(reinterpret_cast<uint2*>(words)), parent(words + 2 * (size_t)n), first(parent + n), owners(first + n),
          sums(owners + n + 1) {}
};
}  // namespace

// Ranges, parents and record numbers of the internal nodes of n >= 2 lights
// with the given sorted codes; out[0] = owners, out[1] = depth (both zeroed by
// the caller).
extern "C" hipError_t hrr_dev_nodes(const uint64_t* code, uint32_t n, uint32_t leaf, uint32_t pow2, uint32_t* words,
                                    uint32_t* out, hipStream_t stream) {
    const NodeTables T(words, n);
    hipError_t e = hipMemsetAsync(T.owners, 0, ((size_t)n + 1) * sizeof(uint32_t), stream);
    if (e != hipSuccess) return e;
    nodes_kernel<<<blocks_for(n - 1), kThreads, 0, stream>>>(code, n, leaf, pow2, T.range, T.parent, T.owners);
    if ((e = scan::exclusive_sum(T.owners, T.owners, n + 1u, T.sums, stream)) != hipSuccess) return e;
    ranks_kernel<<<blocks_for(n - 1), kThreads, 0, stream>>>(T.range, T.parent, T.owners, n, leaf, T.first, out);
    return hipGetLastError();
}

// The records of those nodes (zeroed by the caller where no node writes).
extern "C" hipError_t hrr_dev_records(const uint32_t* words, uint32_t n, const float* lights, const float* blocks,
                                      Node* nodes, hipStream_t stream) {
    const NodeTables T(const_cast<uint32_t*>(words), n);
    records_kernel<<<blocks_for(n - 1), kThreads, 0, stream>>>(
        T.range, T.parent, T.first, reinterpret_cast<const float4*>(lights), reinterpret_cast<const float4*>(blocks),
        block_tree_log(n), n, nodes);
    return hipGetLastError();
}
