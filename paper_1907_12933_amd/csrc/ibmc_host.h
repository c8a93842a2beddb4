// Host-side structures of the library (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <utility>
#include <string>
#include <vector>
#include <deque>

#include "ibmc_internal.h"
#include "kernels_q8.h"
#include "kernels_f32.h"
#include "kernels_cov.h"
#include "kernels_prop.h"
#include "kernels_sort.h"
#include "kernels_lane.h"
#include "kernels_fold.h"

namespace ibmc {

ibmc_status fail(ibmc_status code, const char *fmt, ...);
const char *last_error();
void clear_error();

#define HIP_OK(expr)                                                                              \
    do {                                                                                          \
        hipError_t _e = (expr);                                                                   \
        if (_e != hipSuccess)                                                                     \
            return ::ibmc::fail(IBMC_E_HIP, "%s:%d %s: %s", __FILE__, __LINE__, #expr,             \
                                hipGetErrorString(_e));                                           \
    } while (0)

#define IBMC_TRY(expr)                                                                            \
    do {                                                                                          \
        ibmc_status _s = (expr);                                                                  \
        if (_s < 0) return _s;                                                                    \
    } while (0)

// A fixed region of device memory that buffers are carved from, in order,
// instead of being allocated (the allocation-free entry point).  While one is
// installed on the calling thread, DevBuf::reserve takes its bytes from it and
// fails with a clear error once the region is used up.
struct ScratchArena {
    char *base = nullptr;
    size_t cap = 0;
    size_t used = 0;
};
ScratchArena *&thread_arena();

// Grow-only device allocation (or a view into the thread's arena).
struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
    bool borrowed = false;   // p points into an arena: never freed here
    DevBuf() = default;
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    DevBuf(DevBuf &&o) noexcept : p(o.p), bytes(o.bytes), borrowed(o.borrowed) {
        o.p = nullptr;
        o.bytes = 0;
        o.borrowed = false;
    }
    void swap(DevBuf &o) noexcept {
        std::swap(p, o.p);
        std::swap(bytes, o.bytes);
        std::swap(borrowed, o.borrowed);
    }
    ~DevBuf();
    void release();
    ibmc_status reserve(size_t n);
    ibmc_status upload(const void *src, size_t n, hipStream_t s);
    template <class T> T *as() const { return reinterpret_cast<T *>(p); }
};

// Pinned host memory of one call's uploads and read-backs: pieces are taken in
// order and stay valid until the next call's reset (a call returns with its
// stream idle).  Copies from and to it queue without a wait on the host.  The
// blocks stay until the context goes, kPinKeep bytes at most.  Beyond that, where
// nothing can be pinned, and beyond the blocks at hand while an arena is installed
// (the allocation-free entry point) pageable memory stands in, more slowly.
struct PinPool {
    static constexpr size_t kPinFirst = (size_t)256 << 10;  // the block a context starts with
    static constexpr size_t kPinKeep = (size_t)64 << 20;
    struct Block {
        char *p;
        size_t size, used;
        bool pinned;
    };
    std::vector<Block> blocks;
    PinPool() = default;
    PinPool(const PinPool &) = delete;
    PinPool &operator=(const PinPool &) = delete;
    ~PinPool();
    ibmc_status take(size_t n, void **out);          // 256-byte aligned
    void reset();                                    // every piece is given back, and the pageable memory
};

// Streams of concurrent branches (default priority) with an event each, and the
// event they start from.
struct BranchSet {
    std::vector<hipStream_t> stream;
    std::vector<hipEvent_t> done;
    hipEvent_t fork = nullptr;
    BranchSet() = default;
    BranchSet(const BranchSet &) = delete;
    BranchSet &operator=(const BranchSet &) = delete;
    ~BranchSet();
};

}  // namespace ibmc

struct ibmc_ctx {
    int device = 0;
    int n_cu = 0;
    int arch_major = 0, arch_minor = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    hipEvent_t ev0 = nullptr, ev1 = nullptr, ek0 = nullptr, ek1 = nullptr;
    int32_t *flags_host = nullptr;   // [0] abort request, [1] first hit
    int32_t *flags_dev = nullptr;    // device view of flags_host
    // scratch of the check driver (grow-only)
    ibmc::DevBuf images, props, jobs, u0, prop_ids, counters, recs, ties, order;
    ibmc::DevBuf u0f, sortbuf;
    ibmc::PinPool pin;
    std::map<std::pair<const void *, size_t>, int> occupancy;   // resident workgroups by kernel and LDS bytes
    ibmc::DevBuf train_rows;           // activations and deltas of a training pass (bounded)
    ibmc::DevBuf lut;                  // the table sigmoid's knots (built on first use)
    ibmc::DevBuf fold_in, fold_ws, fold_runs, fold_data;   // folded properties: see run_levels
    ibmc::DevBuf recout;  // sorted records in the public layout, on their way to a host buffer
    ibmc::DevBuf prop_scratch, prop_feat, prop_scores, shell_cum;  // ranked search
    int64_t shell_cum_n = -1, shell_cum_ch = -1;                   // shell_cum holds this plan
    // a ranked search's per-call inputs, packed in pinned host memory and sent
    // to stage_dev in one copy; stage_ev marks that copy's completion
    char *stage_host = nullptr;
    size_t stage_host_bytes = 0;
    ibmc::DevBuf stage_dev;
    hipEvent_t stage_ev = nullptr;
    bool stage_pending = false;
    ibmc::DevBuf cov_img, cov_pots, cov_bits, cov_sums, cov_out;
    // tuned kernel variant per network shape key
    std::map<std::string, std::string> tuned;
    ibmc::BranchSet side;              // of captured batch graphs
    ibmc::BranchSet fold_side;         // of folded launches beside each other
    int64_t graph_launches = 0;
    // the instantiated graph of the last multi-network batch and the
    // signature of every value its launches were captured with
    hipGraphExec_t graph_exec = nullptr;
    std::string graph_sig;
    int64_t graph_reuses = 0;
    bool force_int32_layer1 = false;   // testing aid: take the general first-layer path
    // points of one job of a folded level at most: an aborted check keeps whole
    // jobs (tens of milliseconds each)
    int64_t fold_job_points = (int64_t)1 << 31;
    double last_kernel_seconds = 0.0;
    int last_kernel_launches = 0;
    ~ibmc_ctx();
};

struct ibmc_mlp {
    const uint64_t id = next_id();     // of this load, never used again (an address may be)
    ibmc_ctx *ctx = nullptr;
    int device = -1;
    int act = 0;
    int L = 0;
    std::vector<int> dims;
    std::vector<int> shift;
    std::vector<std::vector<int8_t>> Wq;
    std::vector<std::vector<int32_t>> bq;
    std::vector<std::vector<float>> Wf;
    std::vector<std::vector<float>> bf;
    std::deque<ibmc::DevBuf> buf;      // device copies (stable addresses)
    ibmc::QNetDev qd;
    ibmc::FwdExtra fx;
    ibmc::FNetDev fd;
    ibmc::LaneNetDev lane{};           // integer nets the lane kernels serve (lane.ok)
    int64_t pot_bound[IBMC_MAX_LAYERS + 1] = {};  // integer nets: no potential of layer l is larger in magnitude
    bool fold_ok = false;              // integer nets whose properties may be folded
    bool fold_joint = false;           // their first two layers hold no weight of -128
    std::string forced_variant;
    static uint64_t next_id();
    ~ibmc_mlp();
};

namespace ibmc {
std::string shape_key(const ibmc_mlp *m);
// Resident 256-thread workgroups per compute unit of a kernel at `lds` bytes of
// dynamic LDS, asked once per context.
ibmc_status resident_blocks(ibmc_ctx *ctx, const void *fn, size_t lds, int *occ);
PropParams prop_views(const ibmc_proposer *p);
const EnumVariant *pick_variant(ibmc_ctx *ctx, const ibmc_mlp *net);
bool use_lane(ibmc_ctx *ctx, const ibmc_mlp *net, bool allowed);
// ball_r2 (nullable): per property the squared radius of the L2-ball domain,
// or -1 for its delta set.
ibmc_status check_batch_impl(ibmc_ctx *ctx, const ibmc_property *props, int32_t n_props, const ibmc_check_opts *o,
                             ibmc_check_summary *outs, ibmc_cex *cex_buf, ibmc_cex *tie_buf, bool images_on_device,
                             const int64_t *ball_r2 = nullptr);
// Looks up, once per device and with that device current, the address of
// the allocation-free entry point's fixed scratch array.
ibmc_status noalloc_setup(int device);
}
