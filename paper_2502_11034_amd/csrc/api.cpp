// Host side of libadagc: context, argument validation, per-step scalar preparation and
// kernel sequencing.  See include/adagc.h for the contract of every entry point.

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <utility>
#include <vector>

#include "adagc_internal.h"
#include "muon_internal.h"

using namespace adagc;

struct adagc_ctx {
    int          device = 0;
    int64_t      n_tensors = 0;
    int64_t      n_chunks = 0;
    int64_t      total_elems = 0;
    adagc_config cfg{};
    int          grid_norm = 0;     // workgroups of the norm kernel
    int          grid_update = 0;   // workgroups of the update kernel
    int64_t      n_items = 0;       // its work items, a workgroup for each unless the caller or the device limits them
    int          unroll = 0;
    int          nontemporal = 0;
    int          items_per_chunk = 1;   // work items of the update kernel per chunk
    bool         stream_grads = false;  // the norm kernel reads past the memory-side cache
    bool         small_list = false;    // the per-tensor rule goes into the update kernel (FusedRule)
    Exchange     exchange{};            // and the norms too, in a single launch: possible if its words are there,
    bool         one_launch = false;    // and where it pays

    // A run of tensors with a work table of its own (kGroupBytes)
    struct TensorGroup {
        int64_t     first = 0, count = 0;
        int64_t     elems = 0;
        UpdateItems update{};
        size_t      work_at = 0, items_at = 0;    // its places in the groups' tables
        uint32_t    n_chunks = 0, n_long = 0, n_short = 0, n_tiny = 0;
        int         grid_norm = 0, grid_update = 0;
    };
    std::vector<TensorGroup> tensor_groups;   // empty: the list is stepped as a whole
    const WorkRef* group_work = nullptr;      // device
    const WorkRef* group_items = nullptr;

    std::vector<int64_t>    numel;
    std::vector<int64_t>    chunk_begin;      // n_tensors + 1
    std::vector<void*>      param_copies;     // device pointers, empty until set
    std::vector<TensorArgs> cached_args;      // what the device table currently holds
    std::vector<TensorArgs> scratch_args;     // rebuilt on every step, then compared
    bool                    args_uploaded = false;

    void*        slab = nullptr;              // single device allocation, carved below
    DeviceTables tables{};
    TensorArgs*  d_targs = nullptr;
    // Pinned host mirrors for the asynchronous upload of the pointer table: a ring, so that a caller
    // who alternates between pointer sets (two gradient buffers, say) does not have to wait for the
    // previous upload before the next one can be staged.
    static constexpr int kStagingSlots = 4;
    TensorArgs*  staging = nullptr;           // kStagingSlots consecutive tables, then the read-back area
    char*        readback = nullptr;          // pinned: the device's result arrays as they lie in the slab
    size_t       results_at = 0;              // their place in the slab: norm, coef, flag, and with telemetry the three norms
    size_t       coef_at = 0, flag_at = 0, tele_at = 0;      // relative to the first
    size_t       results_bytes = 0;
    int32_t*     readback_status = nullptr;   // pinned, after the results: the status word of a step with device scalars
    hipEvent_t   upload_done[kStagingSlots] = {nullptr, nullptr, nullptr, nullptr};
    bool         upload_pending[kStagingSlots] = {false, false, false, false};
    uint64_t     uploads = 0;                 // tables uploaded so far; slot = uploads % kStagingSlots
    bool         device_scalars_used = false;   // adagc_step_graph was called: its status word is meaningful

    // Muon (adagc_muon_attach): shapes, the batches the Newton-Schulz iteration runs in (matrices of one padded
    // shape, iterated together by batched launches) and the workspace one batch at a time is carved out of
    struct MuonBatch {
        int mp = 0, np = 0;                  // padded extent of the wide orientation
        std::vector<int64_t> members;        // tensor indices
        int64_t first = 0;                   // place of its first record in muon_matrices
        int64_t apply_blocks = 0;            // the most workgroups that the update of one of them needs
    };
    std::vector<adagc_matrix_shape> shapes;
    std::vector<MuonBatch> muon_batches;
    // Batches that are in the workspace at the same time: their products share launches
    struct MuonRound {
        std::vector<size_t>     batches;     // places in muon_batches
        std::vector<MuonGroup>  groups;      // of the batches, in the same order
        std::vector<MuonLaunch> launches[3]; // by product
    };
    std::vector<MuonRound> muon_rounds;
    MuonMatrix* muon_matrices = nullptr;      // device: the batches' matrices, one batch after another; then the planned launches' arrays
    void*  muon_ws = nullptr;
    size_t muon_ws_bytes = 0;

    std::vector<hipEvent_t> prof_events;      // 4 per step while profiling
    int32_t                 prof_capacity = 0;
    int32_t                 prof_steps = 0;
};

namespace {

struct DeviceGuard {
    int  prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) { ok = false; return; }
        if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
    }
    ~DeviceGuard()
    {
        int cur = -1;
        if (ok && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Largest grid this library launches: the runtime wants workgroups x lanes below 2^32.
constexpr int64_t kMaxGridBlocks = (int64_t)(0xFFFFFFFFu / (uint32_t)kBlock);

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

void free_ctx(adagc_ctx* c)
{
    if (!c) return;
    for (hipEvent_t e : c->prof_events) (void)hipEventDestroy(e);
    for (hipEvent_t e : c->upload_done)
        if (e) (void)hipEventDestroy(e);
    if (c->muon_ws) (void)hipFree(c->muon_ws);
    if (c->muon_matrices) (void)hipFree(c->muon_matrices);
    if (c->staging) (void)hipHostFree(c->staging);
    if (c->slab) (void)hipFree(c->slab);
    delete c;
}

}  // namespace

extern "C" int64_t adagc_chunk_elems(void) { return kChunkElems; }

extern "C" const char* adagc_strerror(int code)
{
    switch (code) {
    case ADAGC_OK: return "ok";
    case ADAGC_ERR_INVALID_ARG: return "invalid argument";
    case ADAGC_ERR_OOM: return "out of memory";
    case ADAGC_ERR_HIP: return "HIP runtime error";
    case ADAGC_ERR_TOO_LARGE: return "tensor list too large (too many chunks or tensors)";
    case ADAGC_ERR_STATE: return "call made in the wrong state";
    default: return "unknown error code";
    }
}

extern "C" int adagc_create(adagc_ctx** out, const adagc_tensor_desc* descs, int64_t n_tensors,
                            const adagc_config* cfg)
{
    if (!out || !descs || !cfg || n_tensors <= 0) return ADAGC_ERR_INVALID_ARG;
    if (cfg->optimizer != ADAGC_OPT_ADAMW && cfg->optimizer != ADAGC_OPT_LION && cfg->optimizer != ADAGC_OPT_MUON)
        return ADAGC_ERR_INVALID_ARG;
    if (cfg->optimizer == ADAGC_OPT_MUON && (cfg->telemetry || cfg->update_clipping)) return ADAGC_ERR_INVALID_ARG;
    if (cfg->grad_dtype != ADAGC_GRAD_F32 && cfg->grad_dtype != ADAGC_GRAD_BF16) return ADAGC_ERR_INVALID_ARG;
    if (cfg->has_bf16_param_copy != 0 && cfg->has_bf16_param_copy != 1) return ADAGC_ERR_INVALID_ARG;
    if (cfg->grid_blocks < 0 || cfg->nontemporal < 0 || cfg->nontemporal > 2 || cfg->schedule < 0 ||
        cfg->schedule_run < 0 || cfg->telemetry < 0 || cfg->telemetry > 1 || cfg->update_clipping < 0 ||
        cfg->update_clipping > 1)
        return ADAGC_ERR_INVALID_ARG;
    if (cfg->unroll != 0 && cfg->unroll != 1 && cfg->unroll != 2 && cfg->unroll != 4) return ADAGC_ERR_INVALID_ARG;
    {
        // unroll*1024-element tiles per chunk, 4096-element ones where the caller leaves unroll to the library (whose own choice
        // depends on the optimizer and on the split and may change; it divides 4, so every such split is whole tiles)
        const int tiles = kVecPerLane / (cfg->unroll ? cfg->unroll : 4);
        static_assert(4 % default_unroll(ADAGC_OPT_ADAMW) == 0 && 4 % default_unroll(ADAGC_OPT_LION) == 0, "see above");
        const int sp = cfg->update_split;
        if (sp < 0 || sp > tiles || (sp & (sp - 1)) != 0) return ADAGC_ERR_INVALID_ARG;
    }
    if (n_tensors > kMaxGridBlocks) return ADAGC_ERR_TOO_LARGE;   // the per-tensor kernels run one workgroup per tensor

    adagc_ctx* c = new (std::nothrow) adagc_ctx;
    if (!c) return ADAGC_ERR_OOM;
    int rc = ADAGC_OK;
    std::vector<uint32_t> chunk_tensor, chunk_index;
    try {
        c->chunk_begin.resize((size_t)n_tensors + 1);
        int64_t n_chunks = 0;
        rc = adagc_build_segment_table(descs, n_tensors, kChunkElems, c->chunk_begin.data(), nullptr,
                                       nullptr, 0, &n_chunks);
        if (rc != ADAGC_OK) { free_ctx(c); return rc; }
        chunk_tensor.resize((size_t)n_chunks);
        chunk_index.resize((size_t)n_chunks);
        rc = adagc_build_segment_table(descs, n_tensors, kChunkElems, c->chunk_begin.data(),
                                       chunk_tensor.data(), chunk_index.data(), n_chunks, &n_chunks);
        if (rc != ADAGC_OK) { free_ctx(c); return rc; }
        c->n_tensors = n_tensors;
        c->n_chunks = n_chunks;
        c->cfg = *cfg;
        c->numel.resize((size_t)n_tensors);
        for (int64_t i = 0; i < n_tensors; ++i) c->numel[(size_t)i] = descs[i].numel;
        c->cached_args.assign((size_t)n_tensors, TensorArgs{});
        c->scratch_args.assign((size_t)n_tensors, TensorArgs{});
    } catch (const std::bad_alloc&) {
        free_ctx(c);
        return ADAGC_ERR_OOM;
    }

    if (hipGetDevice(&c->device) != hipSuccess) {
        free_ctx(c);
        return ADAGC_ERR_HIP;
    }
    // Launch defaults, each chosen by measurement on Llama-3-8B shapes (see the profiles):
    //  - one work item (a chunk in the norm kernel, a tile in the update kernel) per workgroup,
    //    dispatched by the hardware, beat a static persistent grid by 1.5-2 % (a CU that falls
    //    behind simply receives fewer); grid_blocks > 0 selects a persistent grid of that many
    //    workgroups, each walking items b, b+grid, ...
    //  - non-temporal loads/stores in the update kernel: +4.5 %
    //  - visiting order: the list cut into 2 halves, the 4 XCDs that share a half (workgroup b goes
    //    to XCD b mod 8) taking runs of 8 chunks (512 KiB of each fp32 array) in turn.  Against
    //    list order: norm kernel -5 %, update -3.5 %; against 8 parts (one per XCD): update
    //    -1.9 % (AdamW, 8 B parameters), -0.4 % (Lion), -1.2 % (20 001 ragged tensors).  Fewer
    //    address fronts per array mean fewer DRAM rows open at once; runs keep each XCD on
    //    its own pages.
    c->nontemporal = cfg->nontemporal == 2 ? 0 : 1;
    //  - work items of the update kernel: see default_unroll.
    // Both streaming kernels walk their work items b, b+grid, ..., so any grid size is valid.
    for (int64_t i = 0; i < n_tensors; ++i) c->total_elems += descs[i].numel;
    const UpdateItems update = update_items(cfg->optimizer, cfg->unroll, cfg->update_split, cfg->grid_blocks, c->total_elems);
    c->unroll = update.unroll;
    c->items_per_chunk = update.per_chunk;
    auto chunk_len = [&](size_t k) {
        const int64_t rest = c->numel[chunk_tensor[k]] - (int64_t)chunk_index[k] * kChunkElems;
        return rest < kChunkElems ? rest : (int64_t)kChunkElems;
    };
    auto grid_for = [cfg](int64_t items) {
        int64_t want = cfg->grid_blocks > 0 ? (int64_t)cfg->grid_blocks : items;
        if (want > items) want = items;
        return (int)(want > kMaxGridBlocks ? kMaxGridBlocks : want);
    };

    // The chunks in visiting order (see adagc_build_visiting_order): the long ones, then the short and the tiny ones in list
    // order; and the work items of the short ones.  Of chunks `from` to `to`, appended.
    std::vector<WorkRef> work, items, group_work, group_items;
    auto append_range = [&](size_t from, size_t to, std::vector<WorkRef>& to_work, std::vector<WorkRef>& to_items,
                            adagc_ctx::TensorGroup& g) {
        const int per_chunk = g.update.per_chunk, short_items = most_short_items(n_tensors, c->total_elems, per_chunk);
        auto kind_of = [&](size_t k) { return chunk_kind(chunk_len(k), per_chunk, g.update.unroll, short_items); };
        std::vector<uint32_t> longer, order;
        for (size_t k = from; k < to; ++k)
            if (kind_of(k) == kLongChunk) longer.push_back((uint32_t)k);
        order.resize(longer.size());
        int made = ADAGC_OK;
        if (!longer.empty())
            made = adagc_build_visiting_order((int64_t)longer.size(), cfg->schedule ? cfg->schedule : 2,
                                              cfg->schedule_run ? cfg->schedule_run : 8, order.data());
        if (made != ADAGC_OK) return made;
        g.work_at = to_work.size();
        g.items_at = to_items.size();
        auto append = [&](uint32_t k) { to_work.push_back(WorkRef{chunk_tensor[k], k, chunk_index[k], (uint32_t)chunk_len(k)}); };
        for (uint32_t o : order) append(longer[o]);
        for (ChunkKind kind : {kShortChunk, kTinyChunk})
            for (size_t k = from; k < to; ++k) {
                if (kind_of(k) != kind) continue;
                append((uint32_t)k);
                if (kind == kTinyChunk) {
                    ++g.n_tiny;
                    continue;
                }
                for (int part = 0; part < chunk_items(chunk_len(k), per_chunk); ++part) {
                    to_items.push_back(to_work.back());
                    to_items.back().len |= (uint32_t)part << kPartShift;
                }
            }
        g.n_chunks = (uint32_t)(to - from);
        g.n_long = (uint32_t)longer.size();
        g.n_short = (uint32_t)(to_items.size() - g.items_at);
        g.grid_norm = grid_for((int64_t)g.n_chunks - g.n_tiny + (g.n_tiny + 3) / 4);
        g.grid_update = grid_for(count_work_items(g.n_long, g.n_short, g.n_tiny, per_chunk));
        return ADAGC_OK;
    };
    const int64_t grad_bytes = c->total_elems * (cfg->grad_dtype == ADAGC_GRAD_BF16 ? 2 : 4);
    const bool grouped = grad_bytes >= kGroupedBytes && cfg->grid_blocks == 0 && cfg->optimizer != ADAGC_OPT_MUON && c->nontemporal &&
                         !cfg->telemetry;
    adagc_ctx::TensorGroup all;
    try {
        work.reserve(chunk_tensor.size());
        all.update = update;
        rc = append_range(0, chunk_tensor.size(), work, items, all);
        if (rc == ADAGC_OK && grouped) {
            const int64_t most = kGroupBytes / (cfg->grad_dtype == ADAGC_GRAD_BF16 ? 2 : 4);
            group_work.reserve(chunk_tensor.size());
            for (int64_t first = 0; rc == ADAGC_OK && first < n_tensors;) {
                adagc_ctx::TensorGroup g;
                g.first = first;
                first = group_end(descs, n_tensors, first, most);
                g.count = first - g.first;
                for (int64_t i = g.first; i < first; ++i) g.elems += descs[i].numel;
                g.update = update_items(cfg->optimizer, cfg->unroll, cfg->update_split, cfg->grid_blocks, g.elems);
                rc = append_range((size_t)c->chunk_begin[(size_t)g.first], (size_t)c->chunk_begin[(size_t)first], group_work, group_items, g);
                c->tensor_groups.push_back(g);
            }
            if (c->tensor_groups.size() == 1) {           // the list as a whole
                c->tensor_groups.clear();
                group_work.clear();
                group_items.clear();
            }
        }
    } catch (const std::bad_alloc&) { rc = ADAGC_ERR_OOM; }
    if (rc != ADAGC_OK) { free_ctx(c); return rc; }
    const int64_t tiles = count_work_items(all.n_long, all.n_short, all.n_tiny, c->items_per_chunk);

    int64_t most_chunks = 0;
    for (int64_t i = 0; i < n_tensors; ++i) {
        const int64_t n = c->chunk_begin[(size_t)i + 1] - c->chunk_begin[(size_t)i];
        if (n > most_chunks) most_chunks = n;
    }
    c->stream_grads = c->nontemporal && stream_gradients(c->total_elems, cfg->grad_dtype == ADAGC_GRAD_BF16);
    c->small_list = tiles <= fused_max_items(cfg->optimizer, c->items_per_chunk, cfg->grid_blocks) && most_chunks <= kFusedMaxChunks;
    // (with the library's own choice of work items, a workgroup for each)
    const bool one_launch = c->small_list && tiles <= kOneLaunchItems && cfg->grid_blocks == 0 && cfg->optimizer != ADAGC_OPT_MUON &&
                            c->unroll == default_unroll(cfg->optimizer) && c->items_per_chunk == default_items(c->unroll) && c->nontemporal &&
                            !cfg->telemetry;
    if (one_launch) {
        LaunchShape shape{all.n_long, all.n_short, all.n_tiny, 0, most_chunks, true};
        for (int64_t i = 0; i < n_tensors; ++i) {
            shape.n_full += descs[i].numel / kChunkElems;
            shape.alone = shape.alone && descs[i].numel <= kChunkElems / c->items_per_chunk;
        }
        int compute_units = 0;
        if (hipDeviceGetAttribute(&compute_units, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
            free_ctx(c);
            return ADAGC_ERR_HIP;
        }
        c->one_launch = one_launch_pays(cfg->optimizer, cfg->grad_dtype == ADAGC_GRAD_BF16, shape, c->items_per_chunk, compute_units);
    }
    c->grid_norm = all.grid_norm;
    c->n_items = tiles;
    c->grid_update = all.grid_update;

    // One slab, carved into 256-byte aligned arrays.
    const size_t nt = (size_t)n_tensors, nc = (size_t)c->n_chunks;
    size_t off = 0;
    auto carve = [&off](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const size_t o_work = carve(nc * sizeof(WorkRef));
    const size_t o_items = carve(items.size() * sizeof(WorkRef));
    const size_t o_targs = carve(nt * sizeof(TensorArgs));
    const size_t o_partials = carve(nc * sizeof(double));
    const size_t o_sumsq = carve(nt * sizeof(double));
    const size_t o_global = carve(4 * sizeof(double));
    const size_t o_arrivals = carve(sizeof(uint32_t));
    const size_t o_ema_before = carve(nt * sizeof(float));
    const size_t o_scalars = carve(sizeof(StepScalars));
    const size_t o_coef64 = carve(nt * sizeof(double));
    // what adagc_get_norms and adagc_get_state_norms read back, side by side: one copy fetches it
    const size_t o_norm = carve(nt * sizeof(float));
    const size_t o_coef = carve(nt * sizeof(float));
    const size_t o_flag = carve(nt);
    const size_t o_tele_norm = carve(cfg->telemetry ? 3 * nt * sizeof(float) : 0);
    c->results_at = o_norm;
    c->coef_at = o_coef - o_norm;
    c->flag_at = o_flag - o_norm;
    c->tele_at = o_tele_norm - o_norm;
    c->results_bytes = (cfg->telemetry ? o_tele_norm + 3 * nt * sizeof(float) : o_flag + nt) - o_norm;
    const size_t tiles_per_chunk = (size_t)c->items_per_chunk;
    const size_t o_tele_partials = carve(cfg->telemetry ? 3 * nc * tiles_per_chunk * sizeof(double) : 0);
    const size_t o_ustat = carve(cfg->update_clipping ? 2 * nc * tiles_per_chunk * sizeof(double) : 0);
    const size_t o_ucoef64 = carve(cfg->update_clipping ? nt * sizeof(double) : 0);
    const size_t o_words = carve(one_launch ? (2 * nc + nt) * sizeof(uint64_t) : 0);
    const size_t o_launches = carve(one_launch ? (size_t)tiles * kWavesPerBlock * sizeof(uint32_t) : 0);
    const size_t o_group_work = carve(group_work.size() * sizeof(WorkRef));
    const size_t o_group_items = carve(group_items.size() * sizeof(WorkRef));
    const size_t slab_bytes = off;

    hipError_t e = hipMalloc(&c->slab, slab_bytes);
    if (e != hipSuccess) { free_ctx(c); return e == hipErrorOutOfMemory ? ADAGC_ERR_OOM : ADAGC_ERR_HIP; }
    char* base = static_cast<char*>(c->slab);
    if (hipMemset(c->slab, 0, slab_bytes) != hipSuccess) { free_ctx(c); return ADAGC_ERR_HIP; }

    auto upload = [&](size_t to, const std::vector<WorkRef>& from) {
        return from.empty() || hipMemcpy(base + to, from.data(), from.size() * sizeof(WorkRef), hipMemcpyHostToDevice) == hipSuccess;
    };
    if (!upload(o_work, work) || !upload(o_items, items) || !upload(o_group_work, group_work) || !upload(o_group_items, group_items)) {
        free_ctx(c);
        return ADAGC_ERR_HIP;
    }
    c->group_work = reinterpret_cast<const WorkRef*>(base + o_group_work);
    c->group_items = reinterpret_cast<const WorkRef*>(base + o_group_items);
    const size_t staging_bytes = adagc_ctx::kStagingSlots * nt * sizeof(TensorArgs);
    const size_t status_at = staging_bytes + align_up(c->results_bytes, 64);
    if (hipHostMalloc(reinterpret_cast<void**>(&c->staging), status_at + sizeof(int32_t), hipHostMallocDefault) != hipSuccess) {
        free_ctx(c);
        return ADAGC_ERR_HIP;
    }
    c->readback = reinterpret_cast<char*>(c->staging) + staging_bytes;
    c->readback_status = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(c->staging) + status_at);
    for (hipEvent_t& ev : c->upload_done)
        if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
            free_ctx(c);
            return ADAGC_ERR_HIP;
        }

    c->d_targs = reinterpret_cast<TensorArgs*>(base + o_targs);
    DeviceTables& t = c->tables;
    t.work = reinterpret_cast<const WorkRef*>(base + o_work);
    t.items = reinterpret_cast<const WorkRef*>(base + o_items);
    t.targs = c->d_targs;
    t.partials = reinterpret_cast<double*>(base + o_partials);
    t.sumsq = reinterpret_cast<double*>(base + o_sumsq);
    t.global = reinterpret_cast<double*>(base + o_global);
    t.arrivals = reinterpret_cast<uint32_t*>(base + o_arrivals);
    t.ema_before = reinterpret_cast<float*>(base + o_ema_before);
    t.scalars = reinterpret_cast<StepScalars*>(base + o_scalars);
    t.coef64 = reinterpret_cast<double*>(base + o_coef64);
    t.norm = reinterpret_cast<float*>(base + o_norm);
    t.coef = reinterpret_cast<float*>(base + o_coef);
    t.flag = reinterpret_cast<uint8_t*>(base + o_flag);
    t.tele_partials = cfg->telemetry ? reinterpret_cast<double*>(base + o_tele_partials) : nullptr;
    t.tele_norm = cfg->telemetry ? reinterpret_cast<float*>(base + o_tele_norm) : nullptr;
    t.ustat_partials = cfg->update_clipping ? reinterpret_cast<double*>(base + o_ustat) : nullptr;
    t.ucoef64 = cfg->update_clipping ? reinterpret_cast<double*>(base + o_ucoef64) : nullptr;
    if (one_launch) c->exchange = {reinterpret_cast<uint64_t*>(base + o_words), reinterpret_cast<uint32_t*>(base + o_launches), kPolls};
    t.n_chunks = (uint32_t)c->n_chunks;
    t.n_long = all.n_long;
    t.n_short = all.n_short;
    t.n_tiny = all.n_tiny;
    t.n_tensors = (uint32_t)c->n_tensors;

    *out = c;
    return ADAGC_OK;
}

// For tests (not in the header): has the context step in a single launch, whether it pays or not, and sets how often a wave of it looks
// for what others tell before it computes that itself.  False: such a step is not possible.
extern "C" int adagc_internal_set_polls(adagc_ctx* ctx, uint32_t polls)
{
    if (!ctx || !ctx->exchange.words) return 0;
    ctx->one_launch = true;
    ctx->exchange.polls = polls;
    return 1;
}

extern "C" void adagc_destroy(adagc_ctx* ctx)
{
    if (!ctx) return;
    DeviceGuard guard(ctx->device);
    free_ctx(ctx);
}

extern "C" int64_t adagc_num_tensors(const adagc_ctx* ctx) { return ctx ? ctx->n_tensors : ADAGC_ERR_INVALID_ARG; }
extern "C" int64_t adagc_num_chunks(const adagc_ctx* ctx) { return ctx ? ctx->n_chunks : ADAGC_ERR_INVALID_ARG; }

extern "C" int adagc_set_param_copies(adagc_ctx* ctx, void* const* params_bf16)
{
    if (!ctx || !params_bf16) return ADAGC_ERR_INVALID_ARG;
    if (!ctx->cfg.has_bf16_param_copy) return ADAGC_ERR_STATE;
    for (int64_t i = 0; i < ctx->n_tensors; ++i)
        if (!params_bf16[i]) return ADAGC_ERR_INVALID_ARG;
    try {
        ctx->param_copies.assign(params_bf16, params_bf16 + ctx->n_tensors);
    } catch (const std::bad_alloc&) { return ADAGC_ERR_OOM; }
    return ADAGC_OK;
}

namespace {

// Shared front half of the two step entry points: argument checks, per-tensor records, upload of the
// pointer table when it changed.  `capturing` forbids everything but kernel launches.
int prepare_tables(adagc_ctx* ctx, void* const* params, const void* const* grads, void* const* exp_avg,
                   void* const* exp_avg_sq, hipStream_t stream, bool capturing)
{
    const bool adamw = ctx->cfg.optimizer == ADAGC_OPT_ADAMW;
    const bool bf16g = ctx->cfg.grad_dtype == ADAGC_GRAD_BF16;
    const bool copy = ctx->cfg.has_bf16_param_copy != 0;
    if (adamw && !exp_avg_sq) return ADAGC_ERR_INVALID_ARG;
    if (copy && ctx->param_copies.size() != (size_t)ctx->n_tensors) return ADAGC_ERR_STATE;

    // Rebuild the per-tensor records from the caller's pointer arrays.  What follows from them alone, line_offset, is zero in the
    // records that are compared, and worked out for those that are uploaded: most steps find the table as it was.
    const uintptr_t grad_align = bf16g ? 2 : 4;
    for (int64_t i = 0; i < ctx->n_tensors; ++i) {
        TensorArgs& a = ctx->scratch_args[(size_t)i];
        a.param = params[i];
        a.grad = grads[i];
        a.exp_avg = exp_avg[i];
        a.exp_avg_sq = adamw ? exp_avg_sq[i] : nullptr;
        a.param_copy = copy ? ctx->param_copies[(size_t)i] : nullptr;
        if (!a.param || !a.grad || !a.exp_avg || (adamw && !a.exp_avg_sq)) return ADAGC_ERR_INVALID_ARG;
        a.numel = ctx->numel[(size_t)i];
        a.chunk_begin = (uint32_t)ctx->chunk_begin[(size_t)i];
        a.chunk_count = (uint32_t)(ctx->chunk_begin[(size_t)i + 1] - ctx->chunk_begin[(size_t)i]);
        a.vec_ok = (aligned(a.param, 4) && aligned(a.exp_avg, 4) && aligned(a.grad, grad_align) &&
                    (!adamw || aligned(a.exp_avg_sq, 4)) && (!copy || aligned(a.param_copy, 2)))
                       ? 1u : 0u;
        a.line_offset = 0;
    }

    const size_t args_bytes = (size_t)ctx->n_tensors * sizeof(TensorArgs);
    if (!ctx->args_uploaded ||
        std::memcmp(ctx->scratch_args.data(), ctx->cached_args.data(), args_bytes) != 0) {
        if (capturing) return ADAGC_ERR_STATE;   // a recorded copy would re-read the staging buffer on every replay
        // Next slot of the staging ring.  It may still be the source of the upload made kStagingSlots
        // table changes ago; only then (the host that far ahead of the GPU) does this call wait.
        const int slot = (int)(ctx->uploads % adagc_ctx::kStagingSlots);
        if (ctx->upload_pending[slot] && hipEventSynchronize(ctx->upload_done[slot]) != hipSuccess) return ADAGC_ERR_HIP;
        TensorArgs* stage = ctx->staging + (size_t)slot * (size_t)ctx->n_tensors;
        std::memcpy(stage, ctx->scratch_args.data(), args_bytes);
        auto walks = [&](int64_t off_lines) {
            return lines_with_unroll(ctx->cfg.optimizer, ctx->unroll) &&
                   walk_lines(ctx->cfg.optimizer, bf16g, copy, ctx->n_tensors, ctx->total_elems, off_lines, ctx->grid_update, ctx->n_items);
        };
        int64_t off_lines = 0;
        if (walks(ctx->total_elems))             // wherever its tensors start
            for (int64_t i = 0; i < ctx->n_tensors; ++i) {
                stage[i].line_offset = line_offset_of(ctx->scratch_args[(size_t)i]);
                if (stage[i].line_offset) off_lines += ctx->numel[(size_t)i];
            }
        if (hipMemcpyAsync(ctx->d_targs, stage, args_bytes, hipMemcpyHostToDevice, stream) != hipSuccess ||
            hipEventRecord(ctx->upload_done[slot], stream) != hipSuccess)
            return ADAGC_ERR_HIP;
        ctx->tables.off_lines = walks(off_lines);
        ctx->upload_pending[slot] = true;
        ctx->uploads++;
        ctx->cached_args.swap(ctx->scratch_args);
        ctx->args_uploaded = true;
    }
    return ADAGC_OK;
}

}  // namespace

extern "C" int adagc_step(adagc_ctx* ctx, void* const* params, const void* const* grads,
                          void* const* exp_avg, void* const* exp_avg_sq, float* ema_norms,
                          const adagc_hyper* hp, int64_t step, void* stream_v)
{
    if (!ctx || !params || !grads || !exp_avg || !ema_norms || !hp || step < 1) return ADAGC_ERR_INVALID_ARG;
    if (ctx->cfg.optimizer == ADAGC_OPT_MUON) return ADAGC_ERR_STATE;      // stepped with adagc_muon_step
    if (!hyper_ok(*hp, ctx->cfg.optimizer)) return ADAGC_ERR_INVALID_ARG;
    const bool update_clip = hp->clip_mode == ADAGC_MODE_AGC || hp->clip_mode == ADAGC_MODE_CLIPPY;
    if (update_clip && !ctx->cfg.update_clipping) return ADAGC_ERR_STATE;
    const bool bf16g = ctx->cfg.grad_dtype == ADAGC_GRAD_BF16;
    const bool copy = ctx->cfg.has_bf16_param_copy != 0;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    const int rc = prepare_tables(ctx, params, grads, exp_avg, exp_avg_sq, stream, false);
    if (rc != ADAGC_OK) return rc;

    RuleArgs r;
    UpdateArgs u;
    host_step_scalars(*hp, step, r, u);
    FusedRule  rule{};
    Exchange   exchange{};
    ctx->device_scalars_used = false;
    const bool prof = ctx->prof_steps < ctx->prof_capacity;
    hipEvent_t* ev = prof ? &ctx->prof_events[(size_t)ctx->prof_steps * 4] : nullptr;

    if (!prof && !ctx->tensor_groups.empty() && !r.warmup && r.mode == ADAGC_MODE_ADAGC) {       // (profiled steps time the kernels of a whole list)
        for (const adagc_ctx::TensorGroup& g : ctx->tensor_groups) {
            DeviceTables t = ctx->tables;
            t.work = ctx->group_work + g.work_at;
            t.items = ctx->group_items + g.items_at;
            t.n_chunks = g.n_chunks;
            t.n_long = g.n_long;
            t.n_short = g.n_short;
            t.n_tiny = g.n_tiny;
            if (launch_sumsq_partials(t, bf16g, stream_gradients(g.elems, bf16g), g.grid_norm, stream) != hipSuccess ||
                launch_tensor_rules(t, ema_norms, r, (uint32_t)g.first, (uint32_t)g.count, stream) != hipSuccess ||
                launch_update(t, u, ctx->cfg.optimizer, bf16g, copy, g.update.unroll, g.update.per_chunk, ctx->nontemporal, 0, g.grid_update,
                              stream) != hipSuccess)
                return ADAGC_ERR_HIP;
        }
        return ADAGC_OK;
    }
    if (prof && hipEventRecord(ev[0], stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (update_clip) {
        // AGC / Clippy: no gradient norms; the direction's norms (timed in the norm slot together with their
        // per-tensor rule), then the update scales the direction
        if (launch_update_clip_rule(ctx->tables, u, r, ctx->cfg.optimizer, bf16g, ctx->items_per_chunk, ctx->nontemporal,
                                    ctx->grid_update, stream) != hipSuccess)
            return ADAGC_ERR_HIP;
        if (prof && (hipEventRecord(ev[1], stream) != hipSuccess || hipEventRecord(ev[2], stream) != hipSuccess))
            return ADAGC_ERR_HIP;
    } else {
        if (ctx->small_list && !r.warmup && r.mode == ADAGC_MODE_ADAGC) rule = FusedRule{ema_norms, r};
        if (rule.ema && ctx->one_launch && !prof && issues_now(stream)) exchange = ctx->exchange;      // (profiled steps keep a norm kernel to time)
        if (!exchange.words &&
            launch_sumsq_partials(ctx->tables, bf16g, ctx->stream_grads, ctx->grid_norm, stream, nullptr, 0, rule.ema) != hipSuccess)
            return ADAGC_ERR_HIP;
        if (prof && hipEventRecord(ev[1], stream) != hipSuccess) return ADAGC_ERR_HIP;
        if (!rule.ema && launch_rules(ctx->tables, ema_norms, r, stream) != hipSuccess) return ADAGC_ERR_HIP;
        if (prof && hipEventRecord(ev[2], stream) != hipSuccess) return ADAGC_ERR_HIP;
    }
    if (launch_update(ctx->tables, u, ctx->cfg.optimizer, bf16g, copy, ctx->unroll, ctx->items_per_chunk,
                      ctx->nontemporal, ctx->cfg.telemetry, ctx->grid_update, stream, false, rule, exchange) != hipSuccess)
        return ADAGC_ERR_HIP;
    if (prof) {
        if (hipEventRecord(ev[3], stream) != hipSuccess) return ADAGC_ERR_HIP;
        ctx->prof_steps++;
    }
    return ADAGC_OK;
}

extern "C" int adagc_step_graph(adagc_ctx* ctx, void* const* params, const void* const* grads,
                                void* const* exp_avg, void* const* exp_avg_sq, float* ema_norms,
                                const adagc_step_params* step_params, void* stream_v)
{
    if (!ctx || !params || !grads || !exp_avg || !ema_norms || !step_params) return ADAGC_ERR_INVALID_ARG;
    if (ctx->cfg.optimizer == ADAGC_OPT_MUON) return ADAGC_ERR_STATE;
    const bool bf16g = ctx->cfg.grad_dtype == ADAGC_GRAD_BF16;
    const bool copy = ctx->cfg.has_bf16_param_copy != 0;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) return ADAGC_ERR_HIP;
    const bool capturing = cap != hipStreamCaptureStatusNone;
    if (capturing && ctx->prof_capacity > 0) return ADAGC_ERR_STATE;     // event records do not belong in a graph
    const int rc = prepare_tables(ctx, params, grads, exp_avg, exp_avg_sq, stream, capturing);
    if (rc != ADAGC_OK) return rc;

    const bool prof = !capturing && ctx->prof_steps < ctx->prof_capacity;
    hipEvent_t* ev = prof ? &ctx->prof_events[(size_t)ctx->prof_steps * 4] : nullptr;
    ctx->device_scalars_used = true;
    if (prof && hipEventRecord(ev[0], stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (launch_sumsq_partials(ctx->tables, bf16g, ctx->stream_grads, ctx->grid_norm, stream, step_params,
                              ctx->cfg.optimizer) != hipSuccess)
        return ADAGC_ERR_HIP;
    if (prof && hipEventRecord(ev[1], stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (launch_rules(ctx->tables, ema_norms, RuleArgs{}, stream, step_params, ctx->cfg.optimizer) != hipSuccess)
        return ADAGC_ERR_HIP;
    if (prof && hipEventRecord(ev[2], stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (launch_update(ctx->tables, UpdateArgs{}, ctx->cfg.optimizer, bf16g, copy, ctx->unroll, ctx->items_per_chunk,
                      ctx->nontemporal, ctx->cfg.telemetry, ctx->grid_update, stream, true) != hipSuccess)
        return ADAGC_ERR_HIP;
    if (prof) {
        if (hipEventRecord(ev[3], stream) != hipSuccess) return ADAGC_ERR_HIP;
        ctx->prof_steps++;
    }
    return ADAGC_OK;
}

// ---------------------------------------------------------------------------------------------
// Muon

namespace {
constexpr int64_t kMuonTile = 128;     // the matrix-core kernel's block tile: workspace matrices are padded to it
// Matrices of one padded shape are iterated together, up to this many per batched launch and as many as fit this much
// workspace (32 matrices of 4096 x 14336 take 17.2 GB).  32 is where the symmetric products of 4096-row matrices fill
// whole rounds of workgroups: 32 x 136 tiles of 256 x 256 = 17 x 256 compute units.
constexpr int64_t kMuonMaxBatch = 32;
constexpr int64_t kMuonWorkspaceBudget = (int64_t)24 << 30;
inline int64_t pad_to_tile(int64_t x) { return (x + kMuonTile - 1) / kMuonTile * kMuonTile; }
// bf16 elements of workspace per matrix of the largest batch; what a matrix takes of it: X, the next X, A and B.  Batches share it
// as far as it goes.
inline int64_t muon_ws_elems(int64_t mp, int64_t np) { return 4 * mp * np + 2 * mp * mp; }
inline int64_t muon_matrix_elems(int64_t mp, int64_t np) { return 2 * mp * np + 2 * mp * mp; }
}  // namespace

extern "C" int adagc_muon_attach(adagc_ctx* ctx, const adagc_matrix_shape* shapes)
{
    if (!ctx || !shapes) return ADAGC_ERR_INVALID_ARG;
    if (ctx->cfg.optimizer != ADAGC_OPT_MUON || ctx->muon_ws) return ADAGC_ERR_STATE;
    std::vector<adagc_ctx::MuonBatch> groups, batches;
    try {
        for (int64_t i = 0; i < ctx->n_tensors; ++i) {
            const int64_t r = shapes[i].rows, c = shapes[i].cols;
            if (r <= 0 || c <= 0 || r > INT32_MAX || c > INT32_MAX || r * c != ctx->numel[(size_t)i]) return ADAGC_ERR_INVALID_ARG;
            const int64_t mp = pad_to_tile(r < c ? r : c), np = pad_to_tile(r < c ? c : r);
            if (np > INT32_MAX || np / 64 > 65535) return ADAGC_ERR_TOO_LARGE;
            size_t g = 0;
            while (g < groups.size() && (groups[g].mp != mp || groups[g].np != np)) ++g;
            if (g == groups.size()) {
                groups.emplace_back();
                groups[g].mp = (int)mp;
                groups[g].np = (int)np;
            }
            groups[g].members.push_back(i);
        }
        ctx->shapes.assign(shapes, shapes + ctx->n_tensors);
    } catch (const std::bad_alloc&) { return ADAGC_ERR_OOM; }
    DeviceGuard guard(ctx->device);
    if (!guard.ok) {
        ctx->shapes.clear();
        return ADAGC_ERR_HIP;
    }
    // Cut every group into batches of equal size (to one matrix), as large as the limits allow, and allocate the
    // workspace for the largest batch.  If the device cannot give that much, try again with half the batch limit.
    for (int64_t limit = kMuonMaxBatch;; limit /= 2) {
        int64_t ws_elems = 0;
        try {
            batches.clear();
            for (const adagc_ctx::MuonBatch& grp : groups) {
                const int64_t per_matrix = muon_ws_elems(grp.mp, grp.np) * (int64_t)sizeof(uint16_t);
                int64_t cap = kMuonWorkspaceBudget / per_matrix;
                if (cap > limit) cap = limit;
                if (cap < 1) cap = 1;
                const int64_t count = (int64_t)grp.members.size();
                const int64_t n_batches = (count + cap - 1) / cap;
                const int64_t size = (count + n_batches - 1) / n_batches;
                for (int64_t first = 0; first < count; first += size) {
                    const int64_t n = count - first < size ? count - first : size;
                    batches.emplace_back();
                    batches.back().mp = grp.mp;
                    batches.back().np = grp.np;
                    batches.back().members.assign(grp.members.begin() + first, grp.members.begin() + first + n);
                    const int64_t need = n * muon_ws_elems(grp.mp, grp.np);
                    if (need > ws_elems) ws_elems = need;
                }
            }
        } catch (const std::bad_alloc&) {
            ctx->shapes.clear();
            return ADAGC_ERR_OOM;
        }
        const size_t bytes = (size_t)ws_elems * sizeof(uint16_t);
        const hipError_t e = hipMalloc(&ctx->muon_ws, bytes);
        if (e == hipSuccess) {
            ctx->muon_ws_bytes = bytes;
            break;
        }
        ctx->muon_ws = nullptr;
        (void)hipGetLastError();          // the failed allocation is handled here: do not leave its error for the next call
        if (e != hipErrorOutOfMemory || limit == 1) {
            ctx->shapes.clear();
            return e == hipErrorOutOfMemory ? ADAGC_ERR_OOM : ADAGC_ERR_HIP;
        }
    }
    // Rounds: every batch, the largest first, joins the first round with room for it.  Then the records of the matrices, batch by
    // batch, and the planned launches go to device memory.
    int rc = ADAGC_OK;
    std::vector<adagc_ctx::MuonRound> rounds;
    try {
        std::vector<size_t> order(batches.size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = i;
        auto elems = [&](size_t i) { return (int64_t)batches[i].members.size() * muon_matrix_elems(batches[i].mp, batches[i].np); };
        std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return elems(a) > elems(b); });
        std::vector<int64_t> used;
        for (size_t i : order) {
            size_t r = 0;
            while (r < rounds.size() && ((used[r] + elems(i)) * (int64_t)sizeof(uint16_t) > (int64_t)ctx->muon_ws_bytes ||
                                         rounds[r].batches.size() == (size_t)kMaxGroups))
                ++r;
            if (r == rounds.size()) {
                rounds.emplace_back();
                used.push_back(0);
            }
            const adagc_ctx::MuonBatch& bt = batches[i];
            const int64_t n = (int64_t)bt.members.size(), mn = (int64_t)bt.mp * bt.np, mm = (int64_t)bt.mp * bt.mp;
            uint16_t* base = static_cast<uint16_t*>(ctx->muon_ws) + used[r];
            rounds[r].groups.push_back(MuonGroup{bt.mp, bt.np, (int)n, base, base + n * mn, base + 2 * n * mn, base + 2 * n * mn + n * mm});
            rounds[r].batches.push_back(i);
            used[r] += elems(i);
        }
        std::vector<MuonMatrix> records;
        for (adagc_ctx::MuonBatch& bt : batches) {
            bt.first = (int64_t)records.size();
            bt.apply_blocks = 0;
            for (int64_t i : bt.members) {
                const int64_t r = shapes[i].rows, c = shapes[i].cols;
                records.push_back(MuonMatrix{(uint32_t)i, 0u, r, c, std::sqrt(r > c ? (double)r / (double)c : 1.0)});
                bt.apply_blocks = std::max(bt.apply_blocks, muon_apply_blocks(r, c));
            }
        }
        std::vector<GemmItem> items;
        std::vector<int32_t> first;
        std::vector<std::pair<size_t, size_t>> places;            // of a launch's items and first, launch by launch
        for (adagc_ctx::MuonRound& round : rounds) {
            std::vector<MuonExtent> extents;
            for (const MuonGroup& g : round.groups) extents.push_back(MuonExtent{g.mp, g.np, g.count});
            for (int p = 0; p < 3; ++p)
                for (PlannedLaunch& l : plan_muon_product((MuonProduct)p, extents)) {
                    places.emplace_back(items.size(), first.size());
                    items.insert(items.end(), l.items.begin(), l.items.end());
                    first.insert(first.end(), l.first.begin(), l.first.end());
                    round.launches[p].push_back(MuonLaunch{l.side, l.workgroups, l.groups, nullptr, nullptr});
                }
        }
        const size_t records_bytes = records.size() * sizeof(MuonMatrix), items_bytes = items.size() * sizeof(GemmItem);
        const size_t bytes = records_bytes + items_bytes + first.size() * sizeof(int32_t);
        std::vector<char> image(bytes);
        std::memcpy(image.data(), records.data(), records_bytes);
        std::memcpy(image.data() + records_bytes, items.data(), items_bytes);
        std::memcpy(image.data() + records_bytes + items_bytes, first.data(), first.size() * sizeof(int32_t));
        const hipError_t e = hipMalloc(reinterpret_cast<void**>(&ctx->muon_matrices), bytes);
        if (e != hipSuccess) {
            ctx->muon_matrices = nullptr;
            (void)hipGetLastError();
            rc = e == hipErrorOutOfMemory ? ADAGC_ERR_OOM : ADAGC_ERR_HIP;
        } else if (hipMemcpy(ctx->muon_matrices, image.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
            rc = ADAGC_ERR_HIP;
        } else {
            const char* device = reinterpret_cast<const char*>(ctx->muon_matrices);
            const GemmItem* device_items = reinterpret_cast<const GemmItem*>(device + records_bytes);
            const int32_t* device_first = reinterpret_cast<const int32_t*>(device + records_bytes + items_bytes);
            size_t n = 0;
            for (adagc_ctx::MuonRound& round : rounds)
                for (auto& launches : round.launches)
                    for (MuonLaunch& l : launches) {
                        l.items = device_items + places[n].first;
                        l.first = device_first + places[n].second;
                        ++n;
                    }
        }
    } catch (const std::bad_alloc&) { rc = ADAGC_ERR_OOM; }
    if (rc != ADAGC_OK) {                 // as if the call had not been made
        if (ctx->muon_matrices) (void)hipFree(ctx->muon_matrices);
        (void)hipFree(ctx->muon_ws);
        ctx->muon_matrices = nullptr;
        ctx->muon_ws = nullptr;
        ctx->muon_ws_bytes = 0;
        ctx->shapes.clear();
        return rc;
    }
    ctx->muon_rounds.swap(rounds);
    ctx->muon_batches.swap(batches);
    return ADAGC_OK;
}

extern "C" int64_t adagc_muon_workspace_bytes(const adagc_ctx* ctx) { return ctx && ctx->muon_ws ? (int64_t)ctx->muon_ws_bytes : 0; }

extern "C" int adagc_muon_step(adagc_ctx* ctx, void* const* params, const void* const* grads, void* const* momentum,
                               float* ema_norms, const adagc_hyper* hp, const adagc_muon_hyper* mh, int64_t step,
                               void* stream_v)
{
    if (!ctx || !params || !grads || !momentum || !ema_norms || !hp || !mh || step < 1) return ADAGC_ERR_INVALID_ARG;
    if (ctx->cfg.optimizer != ADAGC_OPT_MUON || !ctx->muon_ws) return ADAGC_ERR_STATE;
    adagc_hyper h = *hp;
    h.beta1 = 0.0f;     // Adam's rates and epsilon play no part here; neutral values pass the shared check
    h.beta2 = 0.0f;
    h.eps = 0.0f;
    if (!hyper_ok(h, ADAGC_OPT_LION) || h.clip_mode > ADAGC_MODE_ZCLIP) return ADAGC_ERR_INVALID_ARG;
    if (!(mh->momentum >= 0.0f && mh->momentum < 1.0f) || (mh->nesterov != 0 && mh->nesterov != 1) || mh->ns_steps < 0 ||
        mh->ns_steps > 16 || mh->reserved != 0)
        return ADAGC_ERR_INVALID_ARG;
    const bool bf16g = ctx->cfg.grad_dtype == ADAGC_GRAD_BF16;
    const bool copy = ctx->cfg.has_bf16_param_copy != 0;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    const int rc = prepare_tables(ctx, params, grads, momentum, nullptr, stream, false);
    if (rc != ADAGC_OK) return rc;

    RuleArgs r;
    UpdateArgs u;
    host_step_scalars(h, step, r, u);
    ctx->device_scalars_used = false;
    const bool prof = ctx->prof_steps < ctx->prof_capacity;
    hipEvent_t* ev = prof ? &ctx->prof_events[(size_t)ctx->prof_steps * 4] : nullptr;
    const DeviceTables& t = ctx->tables;

    // gradient norms and clip coefficients: the kernels of adagc_step
    if (prof && hipEventRecord(ev[0], stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (launch_sumsq_partials(t, bf16g, ctx->stream_grads, ctx->grid_norm, stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (prof && hipEventRecord(ev[1], stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (launch_rules(t, ema_norms, r, stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (prof && hipEventRecord(ev[2], stream) != hipSuccess) return ADAGC_ERR_HIP;

    // momentum with the clipped gradient, and ||U||_F^2 of every tensor
    const double mu = (double)mh->momentum;
    if (launch_muon_momentum(t, mu, mh->nesterov, bf16g, ctx->grid_norm, stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (launch_tensor_sumsq(t, stream) != hipSuccess) return ADAGC_ERR_HIP;

    // Newton-Schulz and the update, round by round.
    for (const adagc_ctx::MuonRound& round : ctx->muon_rounds) {
        MuonGroup groups[kMaxGroups];
        const size_t n = round.groups.size();
        std::copy(round.groups.begin(), round.groups.end(), groups);
        MuonSpans spans{};
        for (size_t i = 0; i < n; ++i) {
            const MuonGroup& g = groups[i];
            add_span(spans, ctx->muon_matrices + ctx->muon_batches[round.batches[i]].first, g.x, g.mp, g.np, g.count,
                     muon_normalise_blocks(g.mp, g.np));
        }
        if (launch_muon_normalise(t, spans, mu, mh->nesterov, bf16g, stream) != hipSuccess) return ADAGC_ERR_HIP;
        for (int k = 0; k < mh->ns_steps; ++k) {
            for (int p = 0; p < 3; ++p)
                for (const MuonLaunch& l : round.launches[p])
                    if (launch_muon_product((MuonProduct)p, l, groups, stream) != hipSuccess) return ADAGC_ERR_HIP;
            for (size_t i = 0; i < n; ++i) std::swap(groups[i].x, groups[i].x2);
        }
        spans = MuonSpans{};
        for (size_t i = 0; i < n; ++i) {
            const adagc_ctx::MuonBatch& bt = ctx->muon_batches[round.batches[i]];
            add_span(spans, ctx->muon_matrices + bt.first, groups[i].x, bt.mp, bt.np, groups[i].count, bt.apply_blocks);
        }
        if (launch_muon_apply(t, spans, (double)h.lr, (double)h.weight_decay, copy, stream) != hipSuccess) return ADAGC_ERR_HIP;
    }
    if (prof) {
        if (hipEventRecord(ev[3], stream) != hipSuccess) return ADAGC_ERR_HIP;
        ctx->prof_steps++;
    }
    return ADAGC_OK;
}

namespace {

// The result arrays from byte `from` up to byte `to` (relative to the first) into the read-back area, in one copy to pinned
// memory: a copy to pageable memory waits for the GPU by itself, so that three of them waited three times (GPT-2-small step with
// both read-backs 729 us; now 673.  27 tensors 113, 46).  After adagc_step_graph also the status word that the device wrote for
// that step, to pinned memory as well.
int read_back(adagc_ctx* ctx, size_t from, size_t to, hipStream_t stream)
{
    const char* src = static_cast<const char*>(ctx->slab) + ctx->results_at;
    if (hipMemcpyAsync(ctx->readback + from, src + from, to - from, hipMemcpyDeviceToHost, stream) != hipSuccess) return ADAGC_ERR_HIP;
    const bool status = ctx->device_scalars_used;
    if (status && hipMemcpyAsync(ctx->readback_status, &ctx->tables.scalars->status, sizeof(int32_t), hipMemcpyDeviceToHost,
                                 stream) != hipSuccess)
        return ADAGC_ERR_HIP;
    if (hipStreamSynchronize(stream) != hipSuccess) return ADAGC_ERR_HIP;
    return !status || *ctx->readback_status == 0 ? ADAGC_OK : ADAGC_ERR_INVALID_ARG;
}

}  // namespace

extern "C" int adagc_get_norms(adagc_ctx* ctx, float* host_norms, float* host_coefs, uint8_t* host_clipped,
                               int64_t n_tensors, void* stream_v)
{
    if (!ctx || n_tensors != ctx->n_tensors) return ADAGC_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    const size_t n = (size_t)n_tensors;
    const int rc = read_back(ctx, 0, ctx->flag_at + n, static_cast<hipStream_t>(stream_v));
    if (rc == ADAGC_ERR_HIP) return rc;
    if (host_norms) std::memcpy(host_norms, ctx->readback, n * sizeof(float));
    if (host_coefs) std::memcpy(host_coefs, ctx->readback + ctx->coef_at, n * sizeof(float));
    if (host_clipped) std::memcpy(host_clipped, ctx->readback + ctx->flag_at, n);
    return rc;
}

extern "C" int adagc_get_state_norms(adagc_ctx* ctx, float* host_m_norms, float* host_v_norms,
                                     float* host_update_norms, int64_t n_tensors, void* stream_v)
{
    if (!ctx || n_tensors != ctx->n_tensors) return ADAGC_ERR_INVALID_ARG;
    if (!ctx->cfg.telemetry) return ADAGC_ERR_STATE;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    const size_t n = (size_t)n_tensors;
    const int rc = read_back(ctx, ctx->tele_at, ctx->tele_at + 3 * n * sizeof(float), static_cast<hipStream_t>(stream_v));
    if (rc == ADAGC_ERR_HIP) return rc;
    float* out[3] = {host_m_norms, host_v_norms, host_update_norms};
    for (size_t q = 0; q < 3; ++q)
        if (out[q]) std::memcpy(out[q], ctx->readback + ctx->tele_at + q * n * sizeof(float), n * sizeof(float));
    return rc;
}

extern "C" int adagc_get_segment_table(adagc_ctx* ctx, int64_t* chunk_begin, uint32_t* chunk_tensor,
                                       uint32_t* chunk_index)
{
    if (!ctx) return ADAGC_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    if (chunk_begin) std::memcpy(chunk_begin, ctx->chunk_begin.data(), ((size_t)ctx->n_tensors + 1) * sizeof(int64_t));
    if (chunk_tensor || chunk_index) {
        std::vector<WorkRef> work;
        try {
            work.resize((size_t)ctx->n_chunks);
        } catch (const std::bad_alloc&) { return ADAGC_ERR_OOM; }
        if (hipMemcpy(work.data(), ctx->tables.work, work.size() * sizeof(WorkRef), hipMemcpyDeviceToHost) != hipSuccess)
            return ADAGC_ERR_HIP;
        for (const WorkRef& w : work) {                    // back from visiting order to list order
            if (chunk_tensor) chunk_tensor[w.slot] = w.tensor;
            if (chunk_index) chunk_index[w.slot] = w.index;
        }
    }
    return ADAGC_OK;
}

extern "C" int adagc_profile_begin(adagc_ctx* ctx, int32_t max_steps)
{
    if (!ctx || max_steps <= 0 || max_steps > 4096) return ADAGC_ERR_INVALID_ARG;
    if (!ctx->prof_events.empty()) return ADAGC_ERR_STATE;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    try {
        ctx->prof_events.reserve((size_t)max_steps * 4);
    } catch (const std::bad_alloc&) { return ADAGC_ERR_OOM; }
    for (int32_t k = 0; k < max_steps * 4; ++k) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) {
            for (hipEvent_t x : ctx->prof_events) (void)hipEventDestroy(x);
            ctx->prof_events.clear();
            return ADAGC_ERR_HIP;
        }
        ctx->prof_events.push_back(e);
    }
    ctx->prof_capacity = max_steps;
    ctx->prof_steps = 0;
    return ADAGC_OK;
}

extern "C" int adagc_profile_end(adagc_ctx* ctx, float* ms, int32_t* n_steps)
{
    if (!ctx || !ms || !n_steps) return ADAGC_ERR_INVALID_ARG;
    if (ctx->prof_events.empty()) return ADAGC_ERR_STATE;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ADAGC_ERR_HIP;
    int rc = ADAGC_OK;
    const int32_t n = ctx->prof_steps;
    if (n > 0 && hipEventSynchronize(ctx->prof_events[(size_t)n * 4 - 1]) != hipSuccess) rc = ADAGC_ERR_HIP;
    for (int32_t s = 0; s < n && rc == ADAGC_OK; ++s)
        for (int k = 0; k < 3; ++k)
            if (hipEventElapsedTime(&ms[s * 3 + k], ctx->prof_events[(size_t)s * 4 + k],
                                    ctx->prof_events[(size_t)s * 4 + k + 1]) != hipSuccess)
                rc = ADAGC_ERR_HIP;
    for (hipEvent_t e : ctx->prof_events) (void)hipEventDestroy(e);
    ctx->prof_events.clear();
    ctx->prof_capacity = 0;
    ctx->prof_steps = 0;
    *n_steps = n;
    return rc;
}
