// Shared between the host API and the HIP kernels of libadagc.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "adagc.h"
#include "walk_lines.h"

namespace adagc {

// Elements per chunk.  Every tensor is cut at multiples of this counted from its
// own first element, so a tensor's reduction tree depends only on its own size.
// 16384 fp32 = 64 KiB per stream per chunk: one workgroup of 256 lanes covers a
// full chunk with 16 independent 128-bit loads per lane per stream.
#ifndef ADAGC_CHUNK_ELEMS
#define ADAGC_CHUNK_ELEMS 16384
#endif
constexpr int kChunkElems = ADAGC_CHUNK_ELEMS;
constexpr int kBlock = 256;              // lanes per workgroup (4 wave64)
constexpr int kWavesPerBlock = kBlock / 64;
constexpr int kVecPerLane = kChunkElems / 4 / kBlock;   // 128-bit vectors per lane in a full chunk

// Device-resident per-tensor record: everything a workgroup needs about the
// tensor that owns its chunk, fetched with one scalar load burst.
struct TensorArgs {
    void*       param;       // fp32, in/out
    const void* grad;        // fp32 or bf16, in
    void*       exp_avg;     // fp32, in/out
    void*       exp_avg_sq;  // fp32, in/out (unused by Lion)
    void*       param_copy;  // bf16, out (optional)
    int64_t     numel;
    uint32_t    chunk_begin; // index of this tensor's first chunk / partial slot
    uint32_t    chunk_count;
    uint32_t    vec_ok;      // 1: every pointer is aligned to its elements, which is all that vector accesses need
    uint32_t    line_offset; // elements from a 128-byte line's start to the first element, where param and moments agree on it; else 0
};
static_assert(sizeof(TensorArgs) == 64, "TensorArgs is one 64-byte record");

// TensorArgs::line_offset: the update kernel walks such tensors in whole lines (see there).  The gradient and the copy come along,
// wherever they lie: two of seven arrays, and the copy's and a bf16 gradient's lines hold twice as many elements.
inline uint32_t line_offset_of(const TensorArgs& a)
{
    const auto at = [](const void* p) { return reinterpret_cast<uintptr_t>(p) & 127u; };
    const uintptr_t o = at(a.param);
    return a.vec_ok && at(a.exp_avg) == o && (!a.exp_avg_sq || at(a.exp_avg_sq) == o) ? (uint32_t)(o / 4) : 0u;
}

// One chunk, in the order in which the streaming kernels visit them: all that a workgroup needs to find its elements
// besides the tensor's own record, in one 16-byte load.
// Or one work item of it: the item's number inside the chunk in the upper half of `len`.
struct WorkRef {
    uint32_t tensor;  // owning tensor
    uint32_t slot;    // number in list order: its slot of the partial results
    uint32_t index;   // position inside the tensor: first element = index * kChunkElems
    uint32_t len;     // elements, 1 .. kChunkElems
};
inline constexpr uint32_t kPartShift = 16;
static_assert(kChunkElems < (1 << kPartShift), "a chunk's length and an item's number share a word");

// Scalars of the per-tensor rule (Eq. 3 / warm-up branch of Alg. 1), all widened from the
// caller's fp32 hyper-parameters so that decisions are taken in double.
struct RuleArgs {
    double lambda_rel;
    double ema_beta;
    double lambda_abs;
    double z_thres;      // ZClip
    double lr;           // Clippy's ratio divides by the learning rate
    int    first_step;   // step == 1: gamma is set, not min-ed
    int    warmup;       // step <= t_start
    int    mode;         // ADAGC_MODE_*
    int    pad;
};

// Scalars of the elementwise update, precomputed on the host in double from the caller's fp32
// hyper-parameters.
struct UpdateArgs {
    double beta1, one_minus_beta1;
    double beta2, one_minus_beta2;
    double inv_bias2;      // 1 / (1 - beta2^t)
    double step_size;      // lr / (1 - beta1^t)
    double lr_wd;          // lr * weight_decay
    double eps;
    double lr;             // Lion
    double weight_decay;   // Lion
    double inv_bias1;      // 1 / (1 - beta1^t) (the direction's norms of the update-clipping modes)
    int    update_clip;    // 1: the direction is scaled by the tensor's update coefficient
    int    pad;
};

// Scalars of one step kept in device memory: written by the norm kernel from the caller's
// device-resident adagc_step_params, read by the update kernel.  This is what
// lets a step be recorded into a HIP graph once and replayed for other step numbers.
struct StepScalars {
    UpdateArgs u;
    int32_t    status;   // 0 = valid; otherwise the step leaves all state untouched
    int32_t    pad;
};

struct DeviceTables {
    const WorkRef*    work;       // the chunks in visiting order: the n_long long ones, then the short ones, the n_tiny that one wave
                                  // handles last (chunk_kind)
    const WorkRef*    items;      // the n_short work items of the short chunks
    const TensorArgs* targs;
    double*           partials;   // one per chunk
    double*           sumsq;      // one per tensor
    uint32_t*         arrivals;   // tensors whose sum is stored (model-wide rules); cleared by the norm kernel
    double*           global;     // [0] = model's sum of squares, [1] = its coefficient, [2] = 1 if clipped
    float*            norm;       // per tensor, pre-clip
    float*            coef;       // per tensor, fp32 (reported to the caller)
    double*           coef64;     // per tensor, as computed (what the update kernel multiplies by)
    uint8_t*          flag;       // per tensor, 1 = clip active
    double*           tele_partials;  // telemetry: [3][n_chunks][items per chunk] sums of m^2, v^2, (dtheta)^2 (or null)
    float*            tele_norm;      // telemetry: [3][n_tensors] norms
    StepScalars*      scalars;        // used by adagc_step_graph only
    float*            ema_before;     // per tensor, small lists: gamma as the step found it
    double*           ustat_partials; // update clipping: [2][n_chunks][items per chunk] partial norms of theta and of
                                      // the direction (sums of squares for AGC, maxima for Clippy), or null
    double*           ucoef64;        // update clipping: per-tensor coefficient of the direction, or null
    uint32_t          n_chunks;
    uint32_t          n_long;
    uint32_t          n_short;
    uint32_t          n_tiny;
    uint32_t          n_tensors;
    uint32_t          off_lines;  // host: the update kernel walks whole lines (walk_lines)
};

// Vectors per lane and array that the update kernel keeps in flight, and the work items of a full chunk (one round of those
// each), unless the caller chooses: 2, and items of 2048 elements.  With four waves per SIMD (kUpdateWaves) AdamW has as many loads
// in flight as with 4, items of 4096 and two waves, in smaller pieces, which fill the compute units more evenly and end sooner.
// us per step with 4 and 4096 / with 2 and 2048, tensors of 0.5 to 1.5 M elements: 1.5 M parameters 16.4 / 15.3, 7 M 42.4 / 41.0, 17 M
// 87.8 / 85.9, 64 M 314 / 308, 132 M 661 / 658, 500 M 2642 / 2666, 1.9 G 9306 / 9298; with bf16 gradients and the copy 17.1 / 15.3,
// 46.3 / 44.2, 93.1 / 91.1, 315 / 311, 600 / 591, 2437 / 2434, 8747 / 8755.  In whole chunks a launch has too long a tail and short lists
// too few workgroups.  Lion moves 10 instead of 16 bytes per element each way (Llama-3-8B shapes, 4 layers, two placements, 4 and
// 4096 / 2 and 2048: 7.23 / 6.84 ms, 6.65 / 6.55).
constexpr int default_unroll(int) { return 2; }
constexpr int default_items(int unroll) { return kVecPerLane >= unroll ? kVecPerLane / unroll : 1; }

// What adagc_config's unroll, update_split and grid_blocks (0: the library's choice) make of a list.  Where only the split is chosen, items
// have 4096 elements or more, and AdamW's 4 vectors of each array in flight: us per step with split 4, 2 / 4 vectors: GPT-2-small 654 / 628,
// with bf16 gradients and the copy 620 / 597; 271 M parameters 1434 / 1384, 1372 / 1318.  A workgroup that walks many items has 4 vectors and
// items of 4096 too, as it fetches one after the other: GPT-2-small with 160, 1024 and 16384 workgroups, 2 and 2048 / 4 and 4096: 906 / 762,
// 721 / 691, 662 / 657, bf16 and the copy 991 / 774, 694 / 664, 645 / 625 (320: 784 / 827, 770 / 811; lists of 64 M 444 / 446, 475 / 478).
// The largest launches (elems: the list's, or a group's: see kGroupBytes) have AdamW's 4 vectors and items of 4096.  us per step taken whole, 2 and
// 2048 / 4 and 4096, several placements of the arrays: f32 124 M parameters 616 / 626, 183 M 922 / 930, 238 M 1200 / 1211 and 1215 / 1224,
// 271 M 1374 / 1382 and 1449 / 1433, 354 M 1856 / 1832, 374 M 1975 / 1953 and 1936 / 1931, 423 M 2251 / 2229, 536 M 2828 / 2818,
// 941 M 5300 / 5164; bf16 and the copy 587 / 595, 873 / 880, 1147 / 1157, 1306 / 1312 and 1314 / 1318, 1769 / 1769, 1870 / 1854 and
// 1823 / 1837, 2136 / 2090, 2667 / 2642, 4893 / 4737; in list order (adagc_step_static) 271 M 1351 / 1387, 374 M 1952 / 1947, 423 M 2236 / 2246, 536 M
// 2979 / 2828, 941 M 5041 / 4887.  The smaller items even out a launch, the larger ones open fewer DRAM rows at once.
constexpr int64_t kWideItemsElems = (int64_t)200 << 20;
struct UpdateItems {
    int unroll, per_chunk;
};
constexpr UpdateItems update_items(int optimizer, int unroll, int split, int grid_blocks, int64_t elems)
{
    const int least = default_unroll(optimizer);
    if (unroll == 0) unroll = (split != 0 || grid_blocks != 0 || elems >= kWideItemsElems) && optimizer == ADAGC_OPT_ADAMW ? 4 : least;
    return {unroll, split ? split : default_items(unroll > least ? unroll : least)};
}

// How the streaming kernels work on a chunk of `len` elements, in the order in which the work table has them:
//   long   items_per_chunk work items of the update kernel, numbered with those of other chunks; the last ones may be empty, and an
//          empty workgroup costs its dispatch and a chain of loads all the same
//   short  up to short_items items; the update kernel has a table of them (DeviceTables::items)
//   tiny   one round of a single wave's loads: four chunks to a workgroup.  Most tensors of a list of adapters, biases and norm
//          weights are of this size, and a workgroup of its own for each costs more than its work (5000 tensors, two thirds of
//          them tiny: 108 us per step, now 100).
enum ChunkKind { kLongChunk, kShortChunk, kTinyChunk };
constexpr int kTinyMax = 1024;             // the norm kernel's round for one wave
__host__ __device__ inline int chunk_items(int64_t len, int items_per_chunk)
{
    // = len / (kChunkElems / items_per_chunk) rounded up, without the divisions, which adagc_step_static would have several of per tensor
    return (int)(((uint64_t)len * (uint32_t)items_per_chunk + kChunkElems - 1) / kChunkElems);
}
__host__ __device__ inline ChunkKind chunk_kind(int64_t len, int items_per_chunk, int unroll, int short_items)
{
    if (items_per_chunk == 1 || chunk_items(len, items_per_chunk) > short_items) return kLongChunk;
    return len <= unroll * 256 && len <= kTinyMax ? kTinyChunk : kShortChunk;
}

// The most items of a short chunk.  Half a chunk's in lists of small tensors and in small lists, where empty workgroups are
// what a launch waits for; one elsewhere, because short chunks, visited after the long ones, are far from their neighbours in memory.
// us per step, one / half a chunk's, AdamW with fp32 gradients: 5333 tensors, mean 3000 elements, 122 / 86, 10 666 of them 236 / 164;
// mean 12 000: 4 M parameters 29.6 / 26.8, 16 M 88 / 85, 128 M 664 / 668; mean 30 000: 16 M 83.6 / 80.9, 128 M 642 / 648, 300 M
// 1567 / 1600; mean 200 000: 16 M 85.7 / 83.7.  Lion, bf16: mean 3000: 105 / 74, 209 / 138; mean 30 000: 300 M 1045 / 1052.  (The rule in the
// update kernel, below, has a part in the gain of the lists up to 16 M.)  All chunks that are not full ones short: mean 30 000, 300 M 1621; in
// the order of the long ones, so that their items no longer stay on one XCD: 1669.
constexpr int most_short_items(int64_t n_tensors, int64_t elems, int items_per_chunk)
{
    return items_per_chunk > 1 && (elems <= ((int64_t)32 << 20) || elems < 8192 * n_tensors) ? items_per_chunk / 2 : 1;
}

// Workgroups' worth of work: items_per_chunk for every long chunk (in groups of 8 chunks), those of the short chunks, one for four
// tiny ones.
inline int64_t count_work_items(int64_t n_long, int64_t n_short, int64_t n_tiny, int items_per_chunk)
{
    return (n_long + 7) / 8 * 8 * items_per_chunk + n_short + (n_tiny + 3) / 4;
}

// Whether the norm kernel reads the gradients past the memory-side cache: lists of more than 8 GiB of them, 32 times what
// it holds.  Ordinary loads pay up to about what it holds, from 0.5 to 8 GB the two are within 1 %, at 32 GB streaming ones do
// (figures at the kernel).
inline bool stream_gradients(int64_t total_elems, bool grad_bf16) { return total_elems > ((int64_t)1 << 33) / (grad_bf16 ? 2 : 4); }

// Large lists are stepped group by group (norms, rules, update of one, then of the next) where the rule is per tensor, so that the update
// finds gradients of its group in the memory-side cache: runs of whole tensors of up to so many bytes of gradients, or a
// larger one.
// us per step, whole / in groups, AdamW fp32: 108 M parameters (433 MB of gradients) 535 / 524 in tensors of 1 M, 522 / 531 in tensors of
// 30 000; 133 M 664 / 647, 181 M 908 / 866, 296 M 1533 / 1422; with the copy 1.5 G 7962 / 7319; bf16 and the copy 260 M 1240 / 1206, 583 M
// 2931 / 2669; Lion fp32 108 M 387 / 390, 133 M 483 / 473, 296 M 1075 / 1057, bf16 and the copy 583 M 2005 / 1883.  Groups of 128, 256, 512 and 1024 MiB:
// 1500 ragged tensors of 1.6 GB of gradients 1965, 1905, 1994, 2007 (whole 2039), Llama shapes 9.93, 9.86, 9.95, 10.08 ms (10.22).
constexpr int64_t kGroupBytes = (int64_t)256 << 20, kGroupedBytes = (int64_t)450 << 20;
// Where the group that begins with tensor `first` ends; most: kGroupBytes in elements.  A small tensor before or after one that (nearly) fills a
// group by itself goes with it: three launches and the end of each cost some 10 us, and 16 MiB of gradients from the cache save 3.
// us per step as a whole / small tensors in groups of their own / so, Lion f32: 8 tensors of 70 M elements with one of 4096 after each 2064 / 2073 / 1961,
// 5 with three each 1270 / 1285 / 1204, two of 71 M with two of 1000 each 519 / 524 / 499; AdamW f32 2755 / 2652 / 2414, 1733 / 1677 / 1556,
// 701 / 686 / 661.
inline int64_t group_end(const adagc_tensor_desc* descs, int64_t n_tensors, int64_t first, int64_t most)
{
    int64_t elems = descs[first].numel, largest = elems, end = first + 1;
    for (; end < n_tensors; ++end) {
        const int64_t next = descs[end].numel;
        if (next > largest) largest = next;
        const int64_t with_small = largest + most / 16;
        if (elems + next > (with_small > most ? with_small : most)) break;
        elems += next;
    }
    return end;
}

// Small lists evaluate the per-tensor rule (Eq. 3) inside the update kernel, every wave for its own tensor, from the tensor's
// partial sums and a copy of gamma that the norm kernel makes: one launch less, for one more load per wave.  It needs tensors whose
// slots one wave can sum in the rules kernel's order (see rule_in_update).  us per step, in the rules kernel / in the update, AdamW fp32:
// 0.5 M parameters 12.7 / 9.2, 2 M 18.8 / 16.5, 4 M 28.7 / 26.7, 8 M 48.2 / 46.1, 16 M 83.8 / 81.7, 31 M 156.8 / 155.2; in tensors of 3000:
// 4 M 29.6 / 27.5, 16 M 88.2 / 85.1, 32 M 165.0 / 161.1.  Lion, bf16: 0.5 M 12.5 / 9.1, 4 M 26.4 / 24.4, 16 M 65.1 / 63.5, 31 M 116.1 / 115.3;
// in tensors of 3000: 4 M 25.6 / 24.1, 16 M 73.7 / 73.9, 32 M 137.8 / 140.9.  Work items: about one for 2048 elements.
// (As many fewer of larger items: the line lies at the same list.)  A workgroup that walks many items evaluates the rule for each, one after the
// other: 1024 items where the caller limits the grid.  20 M parameters, in the rules kernel / in the update: AdamW f32 with unroll 4 and 160
// workgroups 113 / 122, Lion with unroll 1 and 320 workgroups 82 / 94, bf16 and the copy 90 / 103.
constexpr int64_t fused_max_items(int optimizer, int items_per_chunk, int grid_blocks)
{
    if (grid_blocks != 0) return 1024;
    return (int64_t)(optimizer == ADAGC_OPT_LION ? 1024 : 2048) * items_per_chunk;
}
constexpr int64_t kFusedMaxChunks = 64;        // of one tensor
struct FusedRule {
    float*   ema;        // null: the rules kernel has run, coefficients are in coef64
    RuleArgs r;
};

// The smallest lists have a single launch: the workgroups of the update kernel sum the chunks for themselves and tell each other
// (Exchange).  Every workgroup of a chunk reads all of its gradient, up to eight times what the norm kernel reads, and waits for the
// others of its tensor, so whether the GPU is done sooner than with two launches depends on the list.  us per step on the GPU, issued
// behind a long product (so the host is ahead), two launches / one:
//                                        AdamW f32    AdamW bf16 + copy   Lion f32     Lion bf16 + copy
//   288 tensors of 2048                  9.0 / 7.3    9.8 / 7.6           7.3 / 5.9    7.7 / 6.5
//   46 of 3693 on average (111 items)    8.3 / 7.5    9.5 / 8.2           7.0 / 7.0    7.8 / 7.6
//   27 of 14 500 (236 items)             9.0 / 8.3    10.9 / 9.5          7.4 / 7.7    8.7 / 8.8
//   12 of 16 384 (128 items)             8.6 / 8.2    9.1 / 9.5           6.6 / 7.5    6.8 / 8.9
//   32 of 16 384 (256 items)             8.7 / 8.6    9.5 / 10.2          7.1 / 8.0    7.3 / 9.8
//   a two-layer transformer (258 items)  8.6 / 8.5    9.5 / 10.1          7.1 / 8.3    7.6 / 9.9
//   17 of 28 200 (275 items)             9.1 / 9.8    11.0 / 10.9         7.8 / 8.4    9.2 / 9.7
//   one tensor of 400 000                8.4 / 8.9    9.4 / 10.7          6.7 / 8.4    7.2 / 10.2
// Where each tensor is one work item nobody waits and nothing is read twice.  Else it pays with AdamW while every workgroup that
// somebody waits for has a compute unit of its own and tensors are not too long; with bf16 gradients not where most long chunks are
// whole ones (two launches take those quickest); with Lion, whose update is short, only without long chunks.  The host saves the issue of
// a launch besides, 2.5 to 3 us.  While a stream is captured there are two launches.
constexpr int64_t kOneLaunchItems = 288;       // of a device with 256 compute units; an eighth more than that on others
constexpr int64_t kOneLaunchChunks = 16;       // of one tensor
struct LaunchShape {
    int64_t n_long, n_short, n_tiny;           // as in DeviceTables
    int64_t n_full;                            // chunks of kChunkElems elements
    int64_t most_chunks;                       // of one tensor
    bool    alone;                             // every tensor is a single work item
};
inline bool one_launch_pays(int optimizer, bool bf16_grads, const LaunchShape& s, int items_per_chunk, int64_t compute_units)
{
    const int64_t items = count_work_items(s.n_long, s.n_short, s.n_tiny, items_per_chunk);
    if (items > kOneLaunchItems || items > compute_units + compute_units / 8) return false;
    if (s.alone) return true;
    if (count_work_items(s.n_long, s.n_short, 0, items_per_chunk) > compute_units) return false;
    if (s.n_long == 0) return true;
    return optimizer == ADAGC_OPT_ADAMW && s.most_chunks <= kOneLaunchChunks && (!bf16_grads || 2 * s.n_full <= s.n_long);
}

// A stream that is being captured (or cannot be asked, as the NULL stream while another one is captured): its launches are issued only once.
// The error of a stream that cannot be asked is not the step's and does not stay behind for the launches, which report the thread's last one.
inline bool issues_now(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// What the workgroups of a launch tell each other: a chunk's sum of squares and a tensor's gamma, in 64-bit words of which the lower
// half is a half of the value and the upper half the launch's number, so that a word is complete by itself and one of an earlier launch is
// not taken for this one's.  Words are stored and loaded with agent-scope accesses (the L2s of the XCDs are not coherent).  Nobody
// waits for long: after `polls` looks a wave computes what it is missing, to the same bits, so that workgroups which are
// not running yet, because other work fills the chip, hold up nothing.
struct Exchange {
    uint64_t* words;         // two for each chunk, then one for each tensor; null: there is a norm kernel
    uint32_t* launches;      // one for each wave, which counts its launches for itself; null: the words are clear, the number is 1
    uint32_t  polls;
};
constexpr uint32_t kPolls = 200;           // a look takes about 1 us

// What every step entry point accepts as hyper-parameters.
inline bool hyper_ok(const adagc_hyper& h, int optimizer)
{
    auto unit = [](float b) { return b >= 0.0f && b < 1.0f; };   // false for NaN
    if (!std::isfinite(h.lr) || !std::isfinite(h.weight_decay)) return false;
    if (!unit(h.beta1) || !unit(h.beta2) || !unit(h.ema_beta)) return false;
    if (optimizer == ADAGC_OPT_ADAMW && !(h.eps >= 0.0f && std::isfinite(h.eps))) return false;
    if (!(h.lambda_rel >= 0.0f)) return false;    // +inf allowed, NaN not
    if (!(h.lambda_abs > 0.0f)) return false;     // +inf allowed, NaN not
    if (h.t_start < 0) return false;
    if (h.clip_mode < ADAGC_MODE_ADAGC || h.clip_mode > ADAGC_MODE_CLIPPY) return false;
    if (h.clip_mode == ADAGC_MODE_ZCLIP && !(h.z_thres > 0.0f)) return false;   // +inf allowed, NaN not
    return true;
}

// Scalars of one step, in double from the caller's fp32 values (host side).
inline void host_step_scalars(const adagc_hyper& hp, int64_t step, RuleArgs& r, UpdateArgs& u)
{
    const double lr = hp.lr, b1 = hp.beta1, b2 = hp.beta2, wd = hp.weight_decay;
    const double t = (double)step;
    r.lambda_rel = (double)hp.lambda_rel;
    r.ema_beta = (double)hp.ema_beta;
    r.lambda_abs = (double)hp.lambda_abs;
    r.z_thres = (double)hp.z_thres;
    r.lr = lr;
    r.pad = 0;
    r.first_step = (step == 1) ? 1 : 0;
    r.warmup = ((step - 1) < (int64_t)hp.t_start) ? 1 : 0;   // steps 1..t_start
    r.mode = hp.clip_mode;
    u.beta1 = b1;
    u.one_minus_beta1 = 1.0 - b1;
    u.beta2 = b2;
    u.one_minus_beta2 = 1.0 - b2;
    u.inv_bias2 = 1.0 / (1.0 - std::pow(b2, t));
    u.step_size = lr / (1.0 - std::pow(b1, t));
    u.lr_wd = lr * wd;
    u.eps = (double)hp.eps;
    u.lr = lr;
    u.weight_decay = wd;
    u.inv_bias1 = 1.0 / (1.0 - std::pow(b1, t));
    u.update_clip = (hp.clip_mode == ADAGC_MODE_AGC || hp.clip_mode == ADAGC_MODE_CLIPPY) ? 1 : 0;
    u.pad = 0;
}

// Launchers (kernels.hip).  Each only enqueues on `stream`.
// Gradient norms, then the clipping rules.  params: null, or the DEVICE parameters of this step, which are then read instead
// of r (and from which the norm kernel leaves t.scalars for launch_update).
hipError_t launch_sumsq_partials(const DeviceTables& t, int grad_bf16, bool streaming, int grid, hipStream_t stream,
                                 const adagc_step_params* params = nullptr, int optimizer = 0, const float* ema_to_keep = nullptr);
hipError_t launch_rules(const DeviceTables& t, float* ema, const RuleArgs& r, hipStream_t stream,
                        const adagc_step_params* params = nullptr, int optimizer = 0);
// The per-tensor rule of tensors first .. first + count - 1 only.
hipError_t launch_tensor_rules(const DeviceTables& t, float* ema, const RuleArgs& r, uint32_t first, uint32_t count, hipStream_t stream);
hipError_t launch_update(const DeviceTables& t, const UpdateArgs& u, int optimizer, int grad_bf16,
                         int with_copy, int unroll, int items_per_chunk, int nt, int tele, int grid,
                         hipStream_t stream, bool device_scalars = false, const FusedRule& rule = FusedRule{}, const Exchange& exchange = Exchange{});
// Update-clipping modes (AGC, Clippy): norms of theta and of the direction per work item, then one workgroup
// per tensor turns them into the tensor's update coefficient.
hipError_t launch_update_clip_rule(const DeviceTables& t, const UpdateArgs& u, const RuleArgs& r, int optimizer,
                                   int grad_bf16, int items_per_chunk, int nt, int grid, hipStream_t stream);
// Per-tensor sums of the per-chunk partials into t.sumsq (K2's fixed order); used by the Muon path for ||U||^2.
hipError_t launch_tensor_sumsq(const DeviceTables& t, hipStream_t stream);

}  // namespace adagc
