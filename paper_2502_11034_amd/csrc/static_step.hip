// adagc_step_static: the step of adagc_step for callers that cannot allocate (code under HIP graph
// capture, tight serving loops, harnesses that forbid hipMalloc).  No context: the segment table,
// the per-chunk partial sums and the per-tensor results live in a fixed array in device memory that
// is part of this library's code object, one copy per GPU, held until the process ends.  The tensor
// records reach the GPU as kernel arguments, so there is no copy, no memset and no event either.
//
// The norm, rule and update kernels are the ones adagc_step launches (kernels.hip), given pointers
// into that array; the chunks are visited in list order, those of one work item after the longer ones.

#include <mutex>

#include "adagc_internal.h"

namespace adagc {
namespace {

constexpr size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Layout of the scratch array (byte offsets, each a multiple of 256).
constexpr size_t kMaxT = ADAGC_STATIC_MAX_TENSORS;
constexpr size_t kMaxC = ADAGC_STATIC_MAX_CHUNKS;
constexpr size_t kOffTargs = 0;
constexpr size_t kOffWork = kOffTargs + align256(kMaxT * sizeof(TensorArgs));
constexpr int kMostShortItems = default_items(default_unroll(ADAGC_OPT_LION)) / 2;         // of a tensor, in its last chunk
constexpr size_t kOffItems = kOffWork + align256(kMaxC * sizeof(WorkRef));
constexpr size_t kOffPartials = kOffItems + align256(kMaxT * kMostShortItems * sizeof(WorkRef));
static_assert(default_items(default_unroll(ADAGC_OPT_ADAMW)) / 2 <= kMostShortItems, "see above");
constexpr size_t kOffSumsq = kOffPartials + align256(kMaxC * sizeof(double));
constexpr size_t kOffCoef64 = kOffSumsq + align256(kMaxT * sizeof(double));
constexpr size_t kOffGlobal = kOffCoef64 + align256(kMaxT * sizeof(double));
constexpr size_t kOffArrivals = kOffGlobal + align256(4 * sizeof(double));
constexpr size_t kOffEmaBefore = kOffArrivals + align256(sizeof(uint32_t));
constexpr size_t kOffNorm = kOffEmaBefore + align256(kMaxT * sizeof(float));
constexpr size_t kOffCoef = kOffNorm + align256(kMaxT * sizeof(float));
constexpr size_t kOffFlag = kOffCoef + align256(kMaxT * sizeof(float));
constexpr size_t kOffWords = kOffFlag + align256(kMaxT);
// of a single launch (Exchange): two for each chunk and one for each tensor, of both up to four for each work item (tiny chunks)
constexpr size_t kMaxWords = (2 + 1) * 4 * kOneLaunchItems;
constexpr size_t kScratchBytes = kOffWords + align256(kMaxWords * sizeof(uint64_t));

// In host code this name is only a handle for hipGetSymbolAddress, never an address to hand to a kernel.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
void*      g_scratch_ptr[kMaxDevices];    // device address of `scratch` on each GPU, once looked up
int        g_compute_units[kMaxDevices];
bool       g_scratch_known[kMaxDevices];
std::mutex g_scratch_mutex;

// Device address of this GPU's copy of the array (`device` must be the current device), and its compute units.
hipError_t scratch_address(int device, unsigned char** out, int* compute_units)
{
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_known[device]) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        e = hipDeviceGetAttribute(&g_compute_units[device], hipDeviceAttributeMultiprocessorCount, device);
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = p;
        g_scratch_known[device] = true;
    }
    *out = static_cast<unsigned char*>(g_scratch_ptr[device]);
    *compute_units = g_compute_units[device];
    return hipSuccess;
}

// Tensor records travel as kernel arguments, a batch per launch: as many as the argument block, 4 KiB, holds.
struct TensorInBatch {
    void*       param;
    const void* grad;
    void*       exp_avg;
    void*       exp_avg_sq;
    void*       param_copy;
    uint64_t    numel;         // and from kVecOkBit and kLineOffsetBit on those two
    uint32_t    chunk_begin;
    uint32_t    long_at;       // where the tensor's long chunks go in the work table, its last chunk if that is no long one, and
    uint32_t    last_at;       // that one's work items if it is a short one
    uint32_t    item_at;
};
constexpr int kBatch = 63, kVecOkBit = 48, kLineOffsetBit = 49;
static_assert(kMaxC * kChunkElems < (size_t)1 << kVecOkBit, "the largest tensor's size leaves the upper bits alone");
struct TensorBatch {
    TensorInBatch t[kBatch];
    uint32_t      first;       // list index of t[0]
    uint32_t      count;
};
static_assert(sizeof(TensorInBatch) == 64 && sizeof(TensorBatch) + 4 * sizeof(void*) + 4 * sizeof(int) <= 4096, "a batch fits the kernel-argument block");

// Workgroup b stores the record of tensor first+b and writes that tensor's rows of the work table.  words: null, or what the
// workgroups of a single launch tell each other, of a list of n_chunks chunks: cleared.
__global__ __launch_bounds__(kBlock) void store_tensor_batch_kernel(TensorBatch batch, TensorArgs* targs, WorkRef* work,
                                                                    WorkRef* items, int items_per_chunk, int unroll, int short_items,
                                                                    uint64_t* words, uint32_t n_chunks)
{
    const uint32_t b = blockIdx.x;
    if (b >= batch.count) return;
    const TensorInBatch& t = batch.t[b];
    const uint32_t i = batch.first + b;
    TensorArgs a;
    a.param = t.param;
    a.grad = t.grad;
    a.exp_avg = t.exp_avg;
    a.exp_avg_sq = t.exp_avg_sq;
    a.param_copy = t.param_copy;
    a.numel = (int64_t)(t.numel & (((uint64_t)1 << kVecOkBit) - 1));
    a.chunk_begin = t.chunk_begin;
    a.chunk_count = (uint32_t)((a.numel + kChunkElems - 1) / kChunkElems);
    a.vec_ok = (uint32_t)(t.numel >> kVecOkBit) & 1u;
    a.line_offset = (uint32_t)(t.numel >> kLineOffsetBit);
    if (threadIdx.x == 0) targs[i] = a;
    if (words) {
        if (threadIdx.x == 0) words[2 * (size_t)n_chunks + i] = 0;
        for (uint32_t k = threadIdx.x; k < 2 * a.chunk_count; k += kBlock) words[2 * (size_t)a.chunk_begin + k] = 0;
    }
    const uint32_t last = a.chunk_count - 1;
    const int64_t last_len = a.numel - (int64_t)last * kChunkElems;
    const ChunkKind last_kind = chunk_kind(last_len, items_per_chunk, unroll, short_items);
    if (last_kind == kShortChunk && (int)threadIdx.x < chunk_items(last_len, items_per_chunk))
        items[t.item_at + threadIdx.x] = WorkRef{i, a.chunk_begin + last, last, (uint32_t)last_len | threadIdx.x << kPartShift};
    for (uint32_t k = threadIdx.x; k < a.chunk_count; k += kBlock) {
        const uint32_t at = k < last || last_kind == kLongChunk ? t.long_at + k : t.last_at;
        work[at] = WorkRef{i, a.chunk_begin + k, k, k < last ? (uint32_t)kChunkElems : (uint32_t)last_len};
    }
}

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

}  // namespace
}  // namespace adagc

using namespace adagc;

extern "C" int adagc_step_static(const adagc_tensor_desc* descs, int64_t n_tensors, const adagc_config* cfg,
                                 void* const* params, const void* const* grads, void* const* exp_avg,
                                 void* const* exp_avg_sq, void* const* params_bf16, float* ema_norms,
                                 const adagc_hyper* hp, int64_t step, float* out_norms, float* out_coefs,
                                 uint8_t* out_clipped, void* stream_v)
{
    if (!descs || !cfg || !params || !grads || !exp_avg || !ema_norms || !hp || n_tensors <= 0 || step < 1)
        return ADAGC_ERR_INVALID_ARG;
    if (cfg->optimizer != ADAGC_OPT_ADAMW && cfg->optimizer != ADAGC_OPT_LION) return ADAGC_ERR_INVALID_ARG;
    if (cfg->grad_dtype != ADAGC_GRAD_F32 && cfg->grad_dtype != ADAGC_GRAD_BF16) return ADAGC_ERR_INVALID_ARG;
    if (cfg->has_bf16_param_copy != 0 && cfg->has_bf16_param_copy != 1) return ADAGC_ERR_INVALID_ARG;
    // no telemetry and no launch tuning here: the defaults, chunks in list order
    if (cfg->telemetry != 0 || cfg->grid_blocks != 0 || cfg->unroll != 0 || cfg->nontemporal != 0 ||
        cfg->schedule != 0 || cfg->update_split != 0 || cfg->schedule_run != 0 || cfg->update_clipping != 0)
        return ADAGC_ERR_INVALID_ARG;
    const bool adamw = cfg->optimizer == ADAGC_OPT_ADAMW;
    const bool bf16g = cfg->grad_dtype == ADAGC_GRAD_BF16;
    const bool copy = cfg->has_bf16_param_copy != 0;
    if (adamw && !exp_avg_sq) return ADAGC_ERR_INVALID_ARG;
    if (copy && !params_bf16) return ADAGC_ERR_INVALID_ARG;
    if (!hyper_ok(*hp, cfg->optimizer) || hp->clip_mode > ADAGC_MODE_ZCLIP) return ADAGC_ERR_INVALID_ARG;
    if (n_tensors > (int64_t)kMaxT) return ADAGC_ERR_TOO_LARGE;

    // Everything is validated before anything is enqueued.
    uint64_t n_chunks = 0, n_long = 0, n_short = 0, n_tiny = 0;          // n_short: work items
    int64_t total_elems = 0, n_full = 0, largest = 0;
    for (int64_t i = 0; i < n_tensors; ++i) {
        if (descs[i].numel <= 0 || descs[i].flags != 0 || descs[i].reserved != 0) return ADAGC_ERR_INVALID_ARG;
        if (!params[i] || !grads[i] || !exp_avg[i] || (adamw && !exp_avg_sq[i]) || (copy && !params_bf16[i]))
            return ADAGC_ERR_INVALID_ARG;
        n_chunks += ((uint64_t)descs[i].numel + kChunkElems - 1) / kChunkElems;
        if (n_chunks > (uint64_t)kMaxC) return ADAGC_ERR_TOO_LARGE;
        if (descs[i].numel > largest) largest = descs[i].numel;
        n_full += (int64_t)((uint64_t)descs[i].numel / kChunkElems);
        total_elems += descs[i].numel;
    }
    const UpdateItems update = update_items(cfg->optimizer, 0, 0, 0, total_elems);
    const int unroll = update.unroll, items_per_chunk = update.per_chunk;
    const int short_items = most_short_items(n_tensors, total_elems, items_per_chunk);
    // the kind of tensor i's last chunk (all others are long)
    auto last_len = [&](int64_t i) { return (int64_t)((uint64_t)(descs[i].numel - 1) % kChunkElems) + 1; };
    auto last_kind = [&](int64_t i) { return chunk_kind(last_len(i), items_per_chunk, unroll, short_items); };
    for (int64_t i = 0; i < n_tensors; ++i) {
        const ChunkKind kind = last_kind(i);
        n_long += (uint64_t)(descs[i].numel - 1) / kChunkElems + (kind == kLongChunk ? 1 : 0);
        n_short += kind == kShortChunk ? (uint64_t)chunk_items(last_len(i), items_per_chunk) : 0;
        n_tiny += kind == kTinyChunk ? 1 : 0;
    }

    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return ADAGC_ERR_HIP;
    if (device < 0 || device >= kMaxDevices) return ADAGC_ERR_HIP;
    unsigned char* base = nullptr;
    int compute_units = 0;
    if (scratch_address(device, &base, &compute_units) != hipSuccess) return ADAGC_ERR_HIP;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);

    DeviceTables t{};
    TensorArgs* d_targs = reinterpret_cast<TensorArgs*>(base + kOffTargs);
    WorkRef* d_work = reinterpret_cast<WorkRef*>(base + kOffWork);
    WorkRef* d_items = reinterpret_cast<WorkRef*>(base + kOffItems);
    t.work = d_work;
    t.items = d_items;
    t.targs = d_targs;
    t.partials = reinterpret_cast<double*>(base + kOffPartials);
    t.sumsq = reinterpret_cast<double*>(base + kOffSumsq);
    t.coef64 = reinterpret_cast<double*>(base + kOffCoef64);
    t.global = reinterpret_cast<double*>(base + kOffGlobal);
    t.arrivals = reinterpret_cast<uint32_t*>(base + kOffArrivals);
    t.ema_before = reinterpret_cast<float*>(base + kOffEmaBefore);
    t.norm = out_norms ? out_norms : reinterpret_cast<float*>(base + kOffNorm);
    t.coef = out_coefs ? out_coefs : reinterpret_cast<float*>(base + kOffCoef);
    t.flag = out_clipped ? out_clipped : reinterpret_cast<uint8_t*>(base + kOffFlag);
    t.tele_partials = nullptr;
    t.tele_norm = nullptr;
    t.scalars = nullptr;
    t.n_chunks = (uint32_t)n_chunks;
    t.n_long = (uint32_t)n_long;
    t.n_short = (uint32_t)n_short;
    t.n_tiny = (uint32_t)n_tiny;
    t.n_tensors = (uint32_t)n_tensors;

    const int64_t items = count_work_items((int64_t)n_long, (int64_t)n_short, (int64_t)n_tiny, items_per_chunk);
    const int64_t max_grid = (int64_t)(0xFFFFFFFFu / (uint32_t)kBlock);
    const int64_t groups = (int64_t)(n_chunks - n_tiny + (n_tiny + 3) / 4);
    const int grid_norm = (int)(groups > max_grid ? max_grid : groups);
    const int grid_update = (int)(items > max_grid ? max_grid : items);

    auto walks = [&](int64_t off_lines) {
        return walk_lines(cfg->optimizer, bf16g, copy, n_tensors, total_elems, off_lines, grid_update, items);
    };
    const bool may_walk = walks(total_elems);        // wherever its tensors start

    RuleArgs r;
    UpdateArgs u;
    host_step_scalars(*hp, step, r, u);
    FusedRule rule{};
    if (largest <= kFusedMaxChunks * kChunkElems && items <= fused_max_items(cfg->optimizer, items_per_chunk, 0) && !r.warmup &&
        r.mode == ADAGC_MODE_ADAGC)
        rule = FusedRule{ema_norms, r};
    const LaunchShape shape{(int64_t)n_long, (int64_t)n_short, (int64_t)n_tiny, n_full, (largest + kChunkElems - 1) / kChunkElems,
                            largest <= kChunkElems / items_per_chunk};
    const bool one_launch = rule.ema && 2 * n_chunks + (uint64_t)n_tensors <= kMaxWords &&
                            one_launch_pays(cfg->optimizer, bf16g, shape, items_per_chunk, compute_units) && issues_now(stream);
    uint64_t* const words = one_launch ? reinterpret_cast<uint64_t*>(base + kOffWords) : nullptr;

    // Tensor records and chunk table, a batch of tensors per launch.
    const uintptr_t grad_align = bf16g ? 2 : 4;
    int64_t off_lines = 0;
    uint32_t chunk_begin = 0, long_at = 0, short_at = (uint32_t)n_long, item_at = 0, tiny_at = (uint32_t)(n_chunks - n_tiny);
    TensorBatch batch;
    for (int64_t first = 0; first < n_tensors; first += kBatch) {
        const int64_t count = (n_tensors - first) < kBatch ? (n_tensors - first) : kBatch;
        for (int64_t b = 0; b < count; ++b) {
            const int64_t i = first + b;
            TensorArgs a{};
            a.param = params[i];
            a.grad = grads[i];
            a.exp_avg = exp_avg[i];
            a.exp_avg_sq = adamw ? exp_avg_sq[i] : nullptr;
            a.param_copy = copy ? params_bf16[i] : nullptr;
            a.vec_ok = (aligned(a.param, 4) && aligned(a.exp_avg, 4) && aligned(a.grad, grad_align) &&
                        (!adamw || aligned(a.exp_avg_sq, 4)) && (!copy || aligned(a.param_copy, 2)))
                           ? 1u : 0u;
            a.line_offset = may_walk ? line_offset_of(a) : 0u;
            if (a.line_offset) off_lines += descs[i].numel;
            const ChunkKind kind = last_kind(i);
            const uint32_t chunks = (uint32_t)(((uint64_t)descs[i].numel + kChunkElems - 1) / kChunkElems);
            batch.t[b] = TensorInBatch{a.param, a.grad, a.exp_avg, a.exp_avg_sq, a.param_copy,
                                       (uint64_t)descs[i].numel | (uint64_t)a.vec_ok << kVecOkBit | (uint64_t)a.line_offset << kLineOffsetBit,
                                       chunk_begin, long_at,
                                       kind == kShortChunk ? short_at++ : (kind == kTinyChunk ? tiny_at++ : 0u), item_at};
            chunk_begin += chunks;
            long_at += kind == kLongChunk ? chunks : chunks - 1;
            if (kind == kShortChunk) item_at += (uint32_t)chunk_items(last_len(i), items_per_chunk);
        }
        for (int64_t b = count; b < kBatch; ++b) batch.t[b] = TensorInBatch{};
        batch.first = (uint32_t)first;
        batch.count = (uint32_t)count;
        store_tensor_batch_kernel<<<dim3((uint32_t)count), dim3(kBlock), 0, stream>>>(batch, d_targs, d_work, d_items,
                                                                                      items_per_chunk, unroll, short_items, words, t.n_chunks);
        if (hipGetLastError() != hipSuccess) return ADAGC_ERR_HIP;
    }

    t.off_lines = walks(off_lines);
    if (!one_launch &&
        launch_sumsq_partials(t, bf16g, stream_gradients(total_elems, bf16g), grid_norm, stream, nullptr, 0, rule.ema) != hipSuccess)
        return ADAGC_ERR_HIP;
    if (!rule.ema && launch_rules(t, ema_norms, r, stream) != hipSuccess) return ADAGC_ERR_HIP;
    if (launch_update(t, u, cfg->optimizer, bf16g, copy, unroll, items_per_chunk, 1, 0, grid_update, stream, false, rule,
                      Exchange{words, nullptr, kPolls}) != hipSuccess)
        return ADAGC_ERR_HIP;
    return ADAGC_OK;
}
