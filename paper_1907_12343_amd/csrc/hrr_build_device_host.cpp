// hrr_build_device_host.cpp -- host driver of the device hierarchy build
// (kernels in hrr_build_device.hip).  The result is the same hierarchy, record
// for record, as hrr_build_hierarchy builds on the host.
#include <hip/hip_runtime_api.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "hrr_ctx.hpp"
#include "hrr_devbuild.hpp"

#define HRR_EXPORT extern "C" __attribute__((visibility("default")))

using hrr::Node;

extern "C" hipError_t hrr_dev_codes(const float* xyz, uint32_t n, const float* qbox, uint64_t* code, uint32_t* idx,
                                    uint32_t* bad, hipStream_t stream);
extern "C" hipError_t hrr_dev_sort(void* temp, size_t* temp_bytes, const uint64_t* code_in, uint64_t* code_out,
                                   const uint32_t* idx_in, uint32_t* idx_out, uint32_t n, hipStream_t stream);
extern "C" hipError_t hrr_dev_gather(const float* xyz, const uint32_t* order, uint32_t n, float* lights,
                                     uint32_t* perm, hipStream_t stream);
extern "C" size_t hrr_dev_nodes_words(uint32_t n);
extern "C" hipError_t hrr_dev_nodes(const uint64_t* code, uint32_t n, uint32_t leaf, uint32_t pow2, uint32_t* words,
                                    uint32_t* out, hipStream_t stream);
extern "C" hipError_t hrr_dev_records(const uint32_t* words, uint32_t n, const float* lights, const float* blocks,
                                      Node* nodes, hipStream_t stream);
extern "C" hipError_t hrr_launch_frontier(const Node* nodes, uint32_t n_lights, uint32_t leaf_size,
                                          const float* blocks, float* out, hipStream_t stream);   // hrr_kernels.hip
extern "C" hipError_t hrr_launch_blocks(const float* lights, uint32_t n_lights, float* blocks, hipStream_t stream);

namespace {

// Carves 256-byte aligned pieces out of one allocation (or, with no base,
// adds up what they need).
struct Carver {
    unsigned char* base;
    size_t at = 0;
    template <typename T>
    T* take(size_t count) {
        T* p = base ? reinterpret_cast<T*>(base + at) : nullptr;
        at += (count * sizeof(T) + 255) / 256 * 256;
        return p;
    }
};

// Build scratch of n lights.
struct Scratch {
    uint32_t* status;   // [0] owners, [1] depth, [2] non-finite coordinate seen
    uint64_t *code_in, *code;
    uint32_t *idx_in, *order, *nodes;
    unsigned char* sort;
    Scratch(Carver& c, uint32_t n, size_t sort_bytes)
        : status(c.take<uint32_t>(8)), code_in(c.take<uint64_t>(n)), code(c.take<uint64_t>(n)),
          idx_in(c.take<uint32_t>(n)), order(c.take<uint32_t>(n)), nodes(c.take<uint32_t>(hrr_dev_nodes_words(n))),
          sort(c.take<unsigned char>(sort_bytes)) {}
};

// Scratch kept between builds is at most this much (2^22 lights need 0.3 GB);
// a larger build gives its own back.
constexpr size_t kKeepScratch = (size_t)512 << 20;

}  // namespace

HRR_EXPORT hrr_status hrr_build_hierarchy_device(hrr_ctx* ctx, const float* lights_xyz_dev, uint32_t n_lights,
                                                 uint32_t leaf_arg, const float* box, void* stream_v,
                                                 hrr_hierarchy** out) {
    using namespace hrr;
    if (!ctx || !out) return fail(HRR_E_INVALID, "hrr_build_hierarchy_device: null argument");
    *out = nullptr;
    if (n_lights > 0 && !lights_xyz_dev) return fail(HRR_E_INVALID, "hrr_build_hierarchy_device: null lights");
    uint32_t leaf_size, split;
    if (!parse_leaf_arg(leaf_arg, &leaf_size, &split))
        return fail(HRR_E_INVALID, "leaf_size must be in [1, 8], optionally with HRR_SPLIT_POW2");
    if (n_lights >= kMaxLights) return fail(HRR_E_INVALID, "at most %u lights", kMaxLights - 1);
    float qbox[6] = {0.f, 0.f, 0.f, 1.f, 1.f, 1.f};
    if (box) {
        for (int k = 0; k < 3; ++k)
            if (!isfinite(box[k]) || !isfinite(box[3 + k]) || !(box[3 + k] > box[k]))
                return fail(HRR_E_INVALID, "box must be finite with hi > lo");
        memcpy(qbox, box, sizeof qbox);
    }
    hipStream_t stream = (hipStream_t)stream_v;
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    const uint32_t n = n_lights;
    const uint32_t max_internal = n > leaf_size ? n - 1 : 0;

    hrr_hierarchy* h = new hrr_hierarchy();
    h->owner = ctx;
    h->n_lights = n;
    h->leaf_size = leaf_size;
    h->split = split;
    struct Building {   // the scratch is in use; one too large to keep is released, on every path
        hrr_ctx* c;
        explicit Building(hrr_ctx* ctx) : c(ctx) {
            std::lock_guard<std::mutex> g(c->build_mu);
            c->building = true;
        }
        ~Building() {
            std::lock_guard<std::mutex> g(c->build_mu);
            c->building = false;
            if (c->build_scratch.bytes > kKeepScratch) c->build_scratch.release();
        }
    } building(ctx);
    auto fail_free = [&](hrr_status st) {
        (void)hipStreamSynchronize(stream);   // the scratch is the context's
        hrr_free_hierarchy(ctx, h);
        return st;
    };
    if (!ctx->build_pin && (e = hipHostMalloc((void**)&ctx->build_pin, 16 * sizeof(uint32_t), hipHostMallocDefault)) != hipSuccess)
        return fail_free(hip_fail(e, "build staging"));
    uint32_t* const pin = ctx->build_pin;

    // everything that is known before the records: one allocation, the records another
    const uint32_t block_log = block_tree_log(n);
    size_t sort_bytes = 0;
    if ((e = hrr_dev_sort(nullptr, &sort_bytes, nullptr, nullptr, nullptr, nullptr, n, stream)) != hipSuccess)
        return fail_free(hip_fail(e, "sort size"));
    Carver size{nullptr};
    (void)Scratch(size, n, sort_bytes);
    if ((e = ctx->build_scratch.ensure(ctx, size.at)) != hipSuccess) return fail_free(hip_fail(e, "build scratch"));
    Carver carve{static_cast<unsigned char*>(ctx->build_scratch.p)};
    const Scratch T(carve, n, sort_bytes);
    const size_t n_block_floats = n ? block_tree_floats(n) : 0;
    const size_t n_frontier_floats = max_internal ? kFrontierWords : 0;
    auto tables = [&](Carver& c) {
        h->d_lights = c.take<float>(std::max<size_t>(n, 1) * 4);
        h->d_perm = c.take<uint32_t>(std::max<size_t>(n, 1));
        float* blocks = c.take<float>(n_block_floats);
        float* frontier = c.take<float>(n_frontier_floats);
        h->d_blocks = n ? blocks : nullptr;
        h->d_frontier = max_internal ? frontier : nullptr;
        if (!max_internal) h->d_nodes = c.take<Node>(1);
    };
    Carver need{nullptr};
    tables(need);
    if ((e = ctx->blocks.get(&h->base, need.at)) != hipSuccess) return fail_free(hip_fail(e, "hierarchy allocation"));
    Carver own{static_cast<unsigned char*>(h->base.p)};
    tables(own);
    h->device_bytes = need.at;

    // 1-3: codes, sort, gather, block tree
    if ((e = hipMemsetAsync(T.status, 0, 8 * sizeof(uint32_t), stream)) != hipSuccess) return fail_free(hip_fail(e, "build"));
    if (n) {
        if ((e = hrr_dev_codes(lights_xyz_dev, n, qbox, T.code_in, T.idx_in, T.status + 2, stream)) != hipSuccess)
            return fail_free(hip_fail(e, "Morton codes"));
        if ((e = hrr_dev_sort(T.sort, &sort_bytes, T.code_in, T.code, T.idx_in, T.order, n, stream)) != hipSuccess)
            return fail_free(hip_fail(e, "sort"));
        if ((e = hrr_dev_gather(lights_xyz_dev, T.order, n, h->d_lights, h->d_perm, stream)) != hipSuccess)
            return fail_free(hip_fail(e, "gather"));
        if ((e = hrr_launch_blocks(h->d_lights, n, h->d_blocks, stream)) != hipSuccess)
            return fail_free(hip_fail(e, "block tree"));
    }
    // 4-5: nodes and record numbers
    if (max_internal && (e = hrr_dev_nodes(T.code, n, leaf_size, split == HRR_SPLIT_POW2 ? 1u : 0u, T.nodes, T.status,
                                           stream)) != hipSuccess)
        return fail_free(hip_fail(e, "nodes"));
    // owners, depth, bad input, and the root box (the block tree's first block)
    float root[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if ((e = hipMemcpyAsync(pin, T.status, 3 * sizeof(uint32_t), hipMemcpyDeviceToHost, stream)) != hipSuccess ||
        (n && (e = hipMemcpyAsync(pin + 4, h->d_blocks + kBlockFloats, sizeof root, hipMemcpyDeviceToHost, stream)) !=
                  hipSuccess) ||
        (e = hipStreamSynchronize(stream)) != hipSuccess)
        return fail_free(hip_fail(e, "device build"));
    if (pin[2]) return fail_free(fail(HRR_E_INVALID, "non-finite light coordinate"));
    if (n) memcpy(root, pin + 4, sizeof root);
    memcpy(h->box, root, 3 * sizeof(float));
    memcpy(h->box + 3, root + 4, 3 * sizeof(float));
    if (max_internal) {
        // 6: the root, the unused record 1, then one sibling pair per owner
        if (pin[0] > max_internal) return fail_free(fail(HRR_E_DEVICE, "device build: record count overflow"));
        const uint32_t n_records = 2u * (1u + pin[0]);
        h->depth = pin[1];
        if ((e = ctx->blocks.get(&h->records, (size_t)n_records * sizeof(Node))) != hipSuccess)
            return fail_free(hip_fail(e, "node records"));
        h->d_nodes = static_cast<Node*>(h->records.p);
        h->n_nodes = n_records;
        h->device_bytes += (size_t)n_records * sizeof(Node);
        if ((e = hipMemsetAsync(h->d_nodes, 0, (size_t)n_records * sizeof(Node), stream)) != hipSuccess ||
            (e = hrr_dev_records(T.nodes, n, h->d_lights, h->d_blocks, h->d_nodes, stream)) != hipSuccess)
            return fail_free(hip_fail(e, "node records"));
        if ((e = hrr_launch_frontier(h->d_nodes, n, leaf_size, h->d_blocks, h->d_frontier, stream)) != hipSuccess ||
            (e = hipMemcpyAsync(pin, h->d_frontier + kFrontierCount, 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, stream)) !=
                hipSuccess ||
            (e = hipStreamSynchronize(stream)) != hipSuccess)
            return fail_free(hip_fail(e, "hierarchy top"));
        h->n_frontier = pin[0];
        memcpy(&h->spread, pin + 1, sizeof h->spread);
    }
    *out = h;
    return HRR_OK;
}
