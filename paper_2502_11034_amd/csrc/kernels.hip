// HIP kernels of libadagc for gfx950 (wave64).
//
//   sumsq_partials_kernel   per chunk:   sum of g^2 in fp64              (l2 norm of Sec. 4.1, for Eq. 3)
//   rules_kernel            per tensor:  norm, h_i, clip flag, EMA update          (Eq. 3, Alg. 1); where one coefficient
//                           serves the whole model, by the workgroup that comes last: warm-up branch of Alg. 1
//                           (GlobalGC + running minimum), GlobalGC on every step (Eq. 2), Global AdaGC (Eq. 3 on the
//                           model's norm; "Ablation Study", Sec. 5.6), ZClip
//   global_rule_kernel / finalize_global_kernel
//                           those model-wide rules on long lists
//   update_kernel           per work item (an eighth of a chunk, a quarter in AdamW's largest launches; chunks of up to 512, 1024,
//                           elements go four to a workgroup): clipped gradient into AdamW / Lion  (Alg. 1); small lists with the
//                           per-tensor rule inside, the smallest with the norms as well
//   tensor_rules_kernel     the per-tensor rule of a group of a large list's tensors
//   direction_stats_kernel / finalize_update_clip_kernel
//                           update clipping (AGC and Clippy rows of Table 2): norms of theta and of the
//                           optimizer's direction per tensor, and the coefficient that scales the direction
//   The norm, rules and update kernels also run with the step's scalars read from device memory, for a launch sequence
//                           that is recorded once and replayed for later steps
//
// Nothing here is a dense contraction, so there is no MFMA: the streaming kernels
// are bound by HBM and are built around 128-bit coalesced accesses with many
// independent loads in flight per lane.  Reductions are deterministic: a lane
// accumulates its elements in index order, lanes are combined with a fixed DPP
// tree, waves through LDS in wave order, chunks by a second kernel in slot order.
// No floating-point atomics anywhere.

#include "adagc_device.h"

namespace adagc {
namespace {

// ---------------------------------------------------------------------------------------------
// wave64 reduction in double: rotate-and-add inside each row of 16 lanes with DPP, then read the
// four row totals with readlane and add them in row order.

template <int DPP_CTRL>
__device__ __forceinline__ double dpp_mov(double x)
{
    int lo = __double2loint(x);
    int hi = __double2hiint(x);
    lo = __builtin_amdgcn_update_dpp(0, lo, DPP_CTRL, 0xF, 0xF, false);
    hi = __builtin_amdgcn_update_dpp(0, hi, DPP_CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double readlane_f64(double x, int lane)
{
    int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
    int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
    return __hiloint2double(hi, lo);
}

// All 64 lanes must be active.  Returns the same value in every lane.
__device__ __forceinline__ double wave_sum_f64(double x)
{
    x += dpp_mov<0x128>(x);  // row_ror:8
    x += dpp_mov<0x124>(x);  // row_ror:4
    x += dpp_mov<0x122>(x);  // row_ror:2
    x += dpp_mov<0x121>(x);  // row_ror:1
    double r0 = readlane_f64(x, 0);
    double r1 = readlane_f64(x, 16);
    double r2 = readlane_f64(x, 32);
    double r3 = readlane_f64(x, 48);
    return ((r0 + r1) + r2) + r3;
}

__device__ __forceinline__ u32x2 pack_bf16x4(f32x4 v)
{
    u32x2 o;
    o.x = float_to_bf16_bits(v.x) | (float_to_bf16_bits(v.y) << 16);
    o.y = float_to_bf16_bits(v.z) | (float_to_bf16_bits(v.w) << 16);
    return o;
}

// ---------------------------------------------------------------------------------------------
// A step whose scalars come from device memory (adagc_step_graph): the step number and the hyper-parameters are read when
// the kernels run, so a recorded launch sequence stays valid for other steps.  Which branch of Alg. 1 applies is therefore
// decided on the device as well.

// The rule's scalars from the caller's step parameters; false if adagc_step would reject those.
__device__ __forceinline__ bool rule_from_params(const adagc_step_params* params, int optimizer, RuleArgs& r)
{
    const adagc_hyper hp = params->hp;
    const int64_t step = params->step;
    auto unit = [](float b) { return b >= 0.0f && b < 1.0f; };   // false for NaN
    auto finite = [](float x) { return fabsf(x) <= 3.402823466e+38f; };
    bool ok = step >= 1 && finite(hp.lr) && finite(hp.weight_decay) && unit(hp.beta1) && unit(hp.beta2) &&
              unit(hp.ema_beta) && hp.lambda_rel >= 0.0f && hp.lambda_abs > 0.0f && hp.t_start >= 0 &&
              hp.clip_mode >= ADAGC_MODE_ADAGC && hp.clip_mode <= ADAGC_MODE_ZCLIP &&
              (hp.clip_mode != ADAGC_MODE_ZCLIP || hp.z_thres > 0.0f);
    if (optimizer == ADAGC_OPT_ADAMW) ok = ok && hp.eps >= 0.0f && finite(hp.eps);
    r.lambda_rel = (double)hp.lambda_rel;
    r.ema_beta = (double)hp.ema_beta;
    r.lambda_abs = (double)hp.lambda_abs;
    r.z_thres = (double)hp.z_thres;
    r.lr = (double)hp.lr;
    r.pad = 0;
    r.first_step = (step == 1) ? 1 : 0;
    r.warmup = ((step - 1) < (int64_t)hp.t_start) ? 1 : 0;
    r.mode = hp.clip_mode;
    return ok;
}

// One lane: validate the caller's step parameters and leave the update kernel's scalars in device memory.
__device__ __forceinline__ void prepare_update_scalars(const DeviceTables& t, const adagc_step_params* params, int optimizer)
{
    RuleArgs r;
    const bool ok = rule_from_params(params, optimizer, r);
    const adagc_hyper hp = params->hp;
    UpdateArgs u;
    const double lr = hp.lr, b1 = hp.beta1, b2 = hp.beta2, wd = hp.weight_decay, tt = (double)params->step;
    u.beta1 = b1;
    u.one_minus_beta1 = 1.0 - b1;
    u.beta2 = b2;
    u.one_minus_beta2 = 1.0 - b2;
    u.inv_bias2 = 1.0 / (1.0 - pow(b2, tt));
    u.step_size = lr / (1.0 - pow(b1, tt));
    u.lr_wd = lr * wd;
    u.eps = (double)hp.eps;
    u.lr = lr;
    u.weight_decay = wd;
    u.inv_bias1 = 1.0 / (1.0 - pow(b1, tt));
    u.update_clip = 0;                          // the update-clipping modes are rejected above
    u.pad = 0;
    t.scalars->u = u;
    t.scalars->status = ok ? 0 : 1;
}

// ---------------------------------------------------------------------------------------------
// K1: one fp64 partial sum of squares per chunk.  Workgroup b takes positions b, b+grid, b+2*grid, ...
// of the visiting order (by default the grid has one workgroup per chunk).

__device__ __forceinline__ void acc4(double (&acc)[4], f32x4 g)
{
    double x = (double)g.x, y = (double)g.y, z = (double)g.z, w = (double)g.w;
    acc[0] = fma(x, x, acc[0]);
    acc[1] = fma(y, y, acc[1]);
    acc[2] = fma(z, z, acc[2]);
    acc[3] = fma(w, w, acc[3]);
}

// Sum of squares of a chunk of at most kTinyMax elements, by one wave (all its lanes get it).
template <bool BF16>
__device__ __forceinline__ double tiny_chunk_sumsq(const gcbytes g, int len, bool vec_ok, int lane)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (vec_ok) {
        constexpr int kRound = kTinyMax / 256;
        const int nvec = len >> 2;
        const int j = (nvec << 2) + lane;
        const float last = j < len ? load_grad1<BF16>(g, j) : 0.f;
        f32x4 r[kRound];
#pragma unroll
        for (int u = 0; u < kRound; ++u) {
            const int v = u * 64 + lane;
            r[u] = v < nvec ? load_grad4<BF16, false>(g, v) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < kRound; ++u) acc4(acc, r[u]);
        const double x = (double)last;
        acc[0] = fma(x, x, acc[0]);
    } else {
        for (int j = lane; j < len; j += 64) {
            const double x = (double)load_grad1<BF16>(g, j);
            acc[0] = fma(x, x, acc[0]);
        }
    }
    return wave_sum_f64((acc[0] + acc[1]) + (acc[2] + acc[3]));
}

// Lane `tid` of a workgroup's share of the sum of squares of any other chunk.
template <bool BF16, bool NTL>
__device__ __forceinline__ double chunk_sumsq_share(const gcbytes g, int len, bool vec_ok, int tid)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (vec_ok) {
        if (len == kChunkElems) {
            f32x4 r[kVecPerLane];
#pragma unroll
            for (int u = 0; u < kVecPerLane; ++u) r[u] = load_grad4<BF16, NTL>(g, u * kBlock + tid);
#pragma unroll
            for (int u = 0; u < kVecPerLane; ++u) acc4(acc, r[u]);
        } else {
            // four loads at a time; a vector past the end counts as zeros, which add nothing to a sum of squares
            constexpr int kFlight = kVecPerLane < 4 ? kVecPerLane : 4;
            const int nvec = len >> 2;
            const int j = (nvec << 2) + tid;
            const float last = j < len ? load_grad1<BF16>(g, j) : 0.f;
            for (int v0 = 0; v0 < nvec; v0 += kFlight * kBlock) {
                f32x4 r[kFlight];
#pragma unroll
                for (int u = 0; u < kFlight; ++u) {
                    const int v = v0 + u * kBlock + tid;
                    r[u] = v < nvec ? load_grad4<BF16, NTL>(g, v) : f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int u = 0; u < kFlight; ++u) acc4(acc, r[u]);
            }
            const double x = (double)last;
            acc[0] = fma(x, x, acc[0]);
        }
    } else {
        for (int j = tid; j < len; j += kBlock) {
            double x = (double)load_grad1<BF16>(g, j);
            acc[0] = fma(x, x, acc[0]);
        }
    }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// NTL: streaming loads, for lists whose gradients are many times the 256 MB of the memory-side cache (stream_gradients).  On
// lists that fit it they would leave nothing there for the update kernel, which reads the same gradients next.  us per step,
// ordinary / streaming loads, with gradients that another kernel writes anew before every step, as a backward pass does:
// 17 MB 31.5 / 33.0, 67 MB 93.6 / 99.4, 268 MB 351 / 374, 266 MB of bf16 647 / 673; then nothing either way beyond 1 %: 498 MB
// 671 / 665, 1.6 GB 2131 / 2123, 3.9 GB of bf16 9.83 / 9.93 ms, 7.7 GB 10.99 / 10.99.  (Where the same gradients are stepped
// again and again, what the cache still holds serves the next step's norms too, and more seems gained than a training step
// has: 498 MB 625 / 655.)  On 32 GB ordinary loads cost this kernel time: 4.49 ms streaming, 4.98 ordinary.
// params: null, or the device-resident parameters of this step, from which one lane makes the update kernel's scalars.
// ema_to_keep: null, or the gammas that the update kernel will need as they are now (see FusedRule).
// One lane also clears the arrival count of the rules kernel.
template <bool BF16, bool NTL>
__global__ __launch_bounds__(kBlock) void sumsq_partials_kernel(DeviceTables t, const adagc_step_params* params, int optimizer,
                                                                const float* ema_to_keep)
{
    __shared__ double wave_sums[kWavesPerBlock];
    const int tid = threadIdx.x;
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        *t.arrivals = 0u;                      // the rules kernel comes next on the stream
        if (params) prepare_update_scalars(t, params, optimizer);
    }

    const uint32_t n_wide = t.n_chunks - t.n_tiny, n_groups = n_wide + (t.n_tiny + 3u) / 4u;
    for (uint32_t k = blockIdx.x; k < n_groups; k += gridDim.x) {
        if (k >= n_wide) {                     // four tiny chunks, one to a wave
            const uint32_t at = n_wide + (k - n_wide) * 4u + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
            if (at < t.n_chunks) {
                const WorkRef w = load_work(t.work, at);
                if (ema_to_keep && w.index == 0 && (tid & 63) == 0) t.ema_before[w.tensor] = ema_to_keep[w.tensor];
                const TensorArgs ta = load_tensor(t.targs, w.tensor);
                const double s = tiny_chunk_sumsq<BF16>(grad_at<BF16>(ta.grad, first_element(w)), (int)w.len, ta.vec_ok != 0, tid & 63);
                if ((tid & 63) == 0) t.partials[w.slot] = s;
            }
            continue;
        }
        const WorkRef w = load_work(t.work, k);
        if (ema_to_keep && w.index == 0 && tid == 0) t.ema_before[w.tensor] = ema_to_keep[w.tensor];
        const TensorArgs ta = load_tensor(t.targs, w.tensor);
        const int len = (int)w.len;
        const gcbytes g = grad_at<BF16>(ta.grad, first_element(w));
        double s = wave_sum_f64(chunk_sumsq_share<BF16, NTL>(g, len, ta.vec_ok != 0, tid));
        if ((tid & 63) == 0) wave_sums[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) {
            double b = wave_sums[0];
#pragma unroll
            for (int v = 1; v < kWavesPerBlock; ++v) b += wave_sums[v];
            t.partials[w.slot] = b;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// K2: per-tensor scalars.  One workgroup per tensor sums that tensor's partial slots in a fixed
// order that depends only on the slot count: lane l owns slots l, l+256, l+512, ... and keeps four
// accumulators (slot row mod 4) so that four loads are in flight; lanes are combined by the
// wave tree, waves through LDS in wave order.

__device__ __forceinline__ double tensor_slot_sum(const DeviceTables& t, const double* slots, uint32_t i,
                                                  double* wave_sums, uint32_t slots_per_chunk = 1)
{
    const uint32_t count = t.targs[i].chunk_count * slots_per_chunk;
    const double* p = slots + (size_t)t.targs[i].chunk_begin * slots_per_chunk;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    uint32_t k = threadIdx.x;
    for (; k + 3 * kBlock < count; k += 4 * kBlock) {
        const double x0 = p[k], x1 = p[k + kBlock], x2 = p[k + 2 * kBlock], x3 = p[k + 3 * kBlock];
        a0 += x0; a1 += x1; a2 += x2; a3 += x3;
    }
    if (k < count) a0 += p[k];
    if (k + kBlock < count) a1 += p[k + kBlock];
    if (k + 2 * kBlock < count) a2 += p[k + 2 * kBlock];
    const double s = wave_sum_f64((a0 + a1) + (a2 + a3));
    if ((threadIdx.x & 63) == 0) wave_sums[threadIdx.x >> 6] = s;
    __syncthreads();
    double total = wave_sums[0];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) total += wave_sums[w];
    return total;
}

// Hand-over between workgroups of one launch.  The L2s of the 8 XCDs are not coherent with each other, so what one
// workgroup leaves for another is written and read with agent-scope accesses, and the count that says so is a release on
// the writer's side and an acquire on the last one's.
template <typename T>
__device__ __forceinline__ T load_shared(const T* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ void store_shared(T* p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One lane: count this workgroup in; true for the last of `total`, which finds everything the others stored before they
// counted themselves.  The counter starts a step at zero because the norm kernel clears it: steps that overlapped by mistake
// leave it at any value, and that must not reach a later one.
__device__ __forceinline__ bool arrive_last(uint32_t* counter, uint32_t total)
{
    if (__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) != total - 1u) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return true;
}

// AdaGC branch of Alg. 1 / Eq. 3 for a tensor with sum of squares s and threshold state gamma_prev, in double, with the
// bits of separately rounded operations: products that are fused are those of fp32 values, which are exact.  (HIP's __dmul_rn and
// __dadd_rn are ordinary operators, which the compiler does fuse, one product of two as it likes: hence the fma.)
struct TensorRule {
    double norm, h, gamma_new;
    bool   active;
};

__device__ __forceinline__ TensorRule adagc_rule(const RuleArgs& r, double s, double gamma_prev)
{
    TensorRule o;
    o.norm = sqrt(s);
    const double threshold = __dmul_rn(r.lambda_rel, gamma_prev);
    o.active = o.norm > threshold;                        // strict; false if either side is NaN
    o.h = o.active ? __ddiv_rn(threshold, o.norm) : 1.0;
    const double clipped_norm = o.active ? threshold : o.norm;
    o.gamma_new = fma(r.ema_beta, gamma_prev, __dmul_rn(__dsub_rn(1.0, r.ema_beta), clipped_norm));
    return o;
}

// One lane: tensor i's results.
__device__ __forceinline__ void store_rule(const DeviceTables& t, float* ema, uint32_t i, double s, const TensorRule& o)
{
    t.sumsq[i] = s;
    t.norm[i] = (float)o.norm;
    t.coef[i] = (float)o.h;
    t.coef64[i] = o.h;
    t.flag[i] = o.active ? 1 : 0;
    ema[i] = (float)o.gamma_new;
}

// Model-wide rules: the model's norm over all tensors (fixed order) and one coefficient for the
// whole model.  Warm-up steps and the GlobalGC mode use Eq. 2; the Global AdaGC mode applies Eq. 3
// (and, during warm-up, the running minimum of Alg. 1) to the model's norm with the single gamma
// kept in ema[0]; the ZClip mode applies Table 2's z-score rule with its mean in ema[0] and its
// variance in ema[1].
__device__ __forceinline__ void global_rule(const DeviceTables& t, float* ema, const RuleArgs& r, double* wave_sums)
{
    const int tid = threadIdx.x;
    double acc = 0.0;
    for (uint32_t i = tid; i < t.n_tensors; i += kBlock) acc += load_shared(t.sumsq + i);
    double s = wave_sum_f64(acc);
    if ((tid & 63) == 0) wave_sums[tid >> 6] = s;
    __syncthreads();
    if (tid != 0) return;
    double total = wave_sums[0];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) total += wave_sums[w];
    const double gnorm = sqrt(total);
    double h;
    bool active, clipped;
    if (r.mode == ADAGC_MODE_GLOBAL_ADAGC && !r.warmup) {
        const double gamma_prev = (double)ema[0];
        const double threshold = __dmul_rn(r.lambda_rel, gamma_prev);
        active = gnorm > threshold;
        h = active ? __ddiv_rn(threshold, gnorm) : 1.0;
        const double clipped_norm = active ? threshold : gnorm;
        ema[0] = (float)fma(r.ema_beta, gamma_prev, __dmul_rn(__dsub_rn(1.0, r.ema_beta), clipped_norm));
        clipped = active;
    } else if (r.mode == ADAGC_MODE_ZCLIP && !r.warmup) {
        // Table 2's ZClip row on the model's norm: z-score against the moving mean and deviation,
        // threshold mu + (z_thres^2 / z) sigma, statistics fed the clipped norm.
        const double mu_prev = (double)ema[0], var_prev = (double)ema[1];
        const double sigma = sqrt(var_prev);
        const double z = __ddiv_rn(__dsub_rn(gnorm, mu_prev), sigma);
        active = z > r.z_thres;                                   // false for NaN (sigma = 0 and norm = mu)
        const double xi = __ddiv_rn(__dmul_rn(r.z_thres, r.z_thres), z);
        const double tau = __dadd_rn(mu_prev, __dmul_rn(xi, sigma));
        h = active ? __ddiv_rn(tau, gnorm) : 1.0;
        const double clipped_norm = active ? tau : gnorm;
        const double mu = fma(r.ema_beta, mu_prev, __dmul_rn(__dsub_rn(1.0, r.ema_beta), clipped_norm));
        const double dev = __dsub_rn(clipped_norm, mu);
        ema[0] = (float)mu;
        ema[1] = (float)fma(r.ema_beta, var_prev, __dmul_rn(__dmul_rn(__dsub_rn(1.0, r.ema_beta), dev), dev));
        clipped = active;
    } else {
        active = gnorm > r.lambda_abs;
        h = active ? __ddiv_rn(r.lambda_abs, gnorm) : 1.0;
        clipped = h < 1.0;
        if (r.mode == ADAGC_MODE_GLOBAL_ADAGC) {
            const double clipped_norm = __dmul_rn(h, gnorm);
            const double gamma_prev = (double)ema[0];
            double gamma_new = clipped_norm;
            if (!r.first_step) gamma_new = clipped_norm < gamma_prev ? clipped_norm : gamma_prev;
            ema[0] = (float)gamma_new;
        }
        if (r.mode == ADAGC_MODE_ZCLIP) {
            // steps that only gather the statistics: set on the first step, moving averages afterwards
            const double clipped_norm = __dmul_rn(h, gnorm);
            double mu = clipped_norm, var = 0.0;
            if (!r.first_step) {
                const double mu_prev = (double)ema[0], var_prev = (double)ema[1];
                mu = fma(r.ema_beta, mu_prev, __dmul_rn(__dsub_rn(1.0, r.ema_beta), clipped_norm));
                const double dev = __dsub_rn(clipped_norm, mu);
                var = fma(r.ema_beta, var_prev, __dmul_rn(__dmul_rn(__dsub_rn(1.0, r.ema_beta), dev), dev));
            }
            ema[0] = (float)mu;
            ema[1] = (float)var;
        }
    }
    t.global[0] = total;
    t.global[1] = h;
    t.global[2] = clipped ? 1.0 : 0.0;
}

// Tensor i under a model-wide rule: it takes the model's coefficient.  In the AdaGC mode (warm-up branch of
// Alg. 1) gamma_i = min{gamma_i, h*n_i}, or h*n_i on the first step; the global modes keep no per-tensor
// state.
__device__ __forceinline__ void take_global_coefficient(const DeviceTables& t, float* ema, const RuleArgs& r, uint32_t i)
{
    const double h = t.global[1];
    const double norm = sqrt(load_shared(t.sumsq + i));
    t.norm[i] = (float)norm;
    t.coef[i] = (float)h;
    t.coef64[i] = h;
    t.flag[i] = (t.global[2] != 0.0) ? 1 : 0;
    if (r.mode == ADAGC_MODE_ADAGC) {
        const double clipped_norm = __dmul_rn(h, norm);
        const double gamma_prev = (double)ema[i];
        double gamma_new = clipped_norm;
        if (!r.first_step) gamma_new = clipped_norm < gamma_prev ? clipped_norm : gamma_prev;
        ema[i] = (float)gamma_new;
    }
}

// Does this step use one coefficient for the whole model?
__device__ __host__ __forceinline__ bool model_wide(const RuleArgs& r) { return r.warmup || r.mode != ADAGC_MODE_ADAGC; }

// K2, one workgroup per tensor.  Per-tensor rule: workgroup i evaluates it.  Model-wide rules on lists of up to kFewTensors
// tensors: the workgroup that stores the last tensor's sum evaluates the rule and hands the coefficient to every tensor, which
// saves two launches and costs the counting, 14 ns a tensor on one address (the release finds the L2 clean here, where next to
// nothing is written; counted in the norm kernel, one release per chunk, it cost half as much again as the whole step).
// us per step with GlobalGC, counted / in two more kernels, tensors of 1000 elements and of 65 536:
//   step         64 tensors 11.9 / 15.2 and 30.2 / 32.7   192: 14.8 / 15.5 and 74.5 / 75.0   256: 15.9 / 15.1 and 93.2 / 91.2
//                512: 20.3 / 15.7 and 173.8 / 169.1
//   graph replay 64 tensors 13.3 / 14.5 and 31.1 / 32.4   192: 15.8 / 14.8 and 75.2 / 76.3   256: 17.4 / 15.0 and 94.2 / 92.7
//                512: 21.3 / 16.1 and 174.6 / 170.7
// (Where a slow host's launches are what a step waits for, counting is ahead up to 300 tensors.)
constexpr uint32_t kFewTensors = 192;

__global__ __launch_bounds__(kBlock) void rules_kernel(DeviceTables t, float* ema, RuleArgs r, const adagc_step_params* params,
                                                       int optimizer)
{
    __shared__ double wave_sums[kWavesPerBlock];
    __shared__ int    last;
    const int tid = threadIdx.x;
    if (params && !rule_from_params(params, optimizer, r)) return;       // the same in all workgroups: nothing is touched
    const uint32_t i = blockIdx.x;
    const double s = tensor_slot_sum(t, t.partials, i, wave_sums);
    if (!model_wide(r)) {
        if (tid == 0) store_rule(t, ema, i, s, adagc_rule(r, s, (double)ema[i]));
        return;
    }
    if (t.n_tensors > kFewTensors) {
        if (tid == 0) t.sumsq[i] = s;
        return;
    }
    if (tid == 0) {
        store_shared(t.sumsq + i, s);
        last = arrive_last(t.arrivals, t.n_tensors) ? 1 : 0;
    }
    __syncthreads();                             // wave_sums is free again as well
    if (!last) return;
    global_rule(t, ema, r, wave_sums);
    __syncthreads();
    for (uint32_t k = tid; k < t.n_tensors; k += kBlock) take_global_coefficient(t, ema, r, k);
}

// The per-tensor rule of a group's tensors, the first of which is `first`.
__global__ __launch_bounds__(kBlock) void tensor_rules_kernel(DeviceTables t, float* ema, RuleArgs r, uint32_t first)
{
    __shared__ double wave_sums[kWavesPerBlock];
    const uint32_t i = first + blockIdx.x;
    const double s = tensor_slot_sum(t, t.partials, i, wave_sums);
    if (threadIdx.x == 0) store_rule(t, ema, i, s, adagc_rule(r, s, (double)ema[i]));
}

// Per-tensor sum of squares only.
__global__ __launch_bounds__(kBlock) void tensor_sumsq_kernel(DeviceTables t)
{
    __shared__ double wave_sums[kWavesPerBlock];
    const uint32_t i = blockIdx.x;
    const double s = tensor_slot_sum(t, t.partials, i, wave_sums);
    if (threadIdx.x == 0) t.sumsq[i] = s;
}

// Model-wide rules on long lists: the rule, then every tensor's share.
__global__ __launch_bounds__(kBlock) void global_rule_kernel(DeviceTables t, float* ema, RuleArgs r, const adagc_step_params* params,
                                                             int optimizer)
{
    __shared__ double wave_sums[kWavesPerBlock];
    if (params && !rule_from_params(params, optimizer, r)) return;
    if (model_wide(r)) global_rule(t, ema, r, wave_sums);                // the same in all lanes
}

__global__ __launch_bounds__(kBlock) void finalize_global_kernel(DeviceTables t, float* ema, RuleArgs r, const adagc_step_params* params,
                                                                 int optimizer)
{
    if (params && !rule_from_params(params, optimizer, r)) return;
    if (!model_wide(r)) return;
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < t.n_tensors) take_global_coefficient(t, ema, r, i);
}

// ---------------------------------------------------------------------------------------------
// K3: clipped gradient into the optimizer, element by element.

struct ElemState {
    float p, m, v;
};

// The elementwise update is evaluated in double and each stored value is rounded to fp32 once.
// The kernel waits on HBM (hardware counters on Llama-3-8B shapes: memory interface busy 99 %,
// vector ALU active 15 % of the time), so double arithmetic costs no time (measured: 37.9 ms with
// either precision) and makes the result the correctly rounded value of Alg. 1's statements, not
// an accumulation of fp32 roundings.
// Every sum of products is written as the fma it is to become: where the compiler may choose which of two products it fuses, it chooses
// differently from kernel to kernel and from element to element of one, and a value then depends (in its last bit, about once in
// 10^9) on where its tensor lies.  beta * state is exact in double (both come from fp32), so fma(beta, state, x) has the bits
// of the separately rounded sum.

// AdamW statements of Alg. 1 on the clipped gradient h*g; the bias corrections are folded into two
// host-computed scalars (step_size = lr / (1 - beta1^t), inv_bias2 = 1 / (1 - beta2^t)).
// uc scales the direction m_hat/(sqrt(v_hat)+eps) (update clipping); it is exactly 1.0 in every other mode.
__device__ __forceinline__ void adamw_elem(const UpdateArgs& a, double h, double uc, float g, ElemState& s)
{
    const double gh = h * (double)g;
    const double m = fma(a.beta1, (double)s.m, a.one_minus_beta1 * gh);
    const double v = fma(a.beta2, (double)s.v, a.one_minus_beta2 * gh * gh);
    const double denom = sqrt(v * a.inv_bias2) + a.eps;
    const double th = (double)s.p;
    s.p = (float)fma(-uc, a.step_size * m / denom, fma(-a.lr_wd, th, th));
    s.m = (float)m;
    s.v = (float)v;
}

// Lion (rule of Chen et al.; the paper only cites it).  The sign is a discrete decision: the
// interpolation c has the bits of the sequence of separately rounded operations that a plain C
// implementation without contraction produces.
__device__ __forceinline__ double lion_sign(const UpdateArgs& a, double gh, float m)
{
    const double c = fma(a.beta1, (double)m, a.one_minus_beta1 * gh);
    return (c > 0.0) ? 1.0 : ((c < 0.0) ? -1.0 : 0.0);
}

__device__ __forceinline__ void lion_elem(const UpdateArgs& a, double h, double uc, float g, ElemState& s)
{
    const double gh = h * (double)g;
    const double sgn = lion_sign(a, gh, s.m);
    const double th = (double)s.p;
    s.p = (float)fma(-a.lr, fma(a.weight_decay, th, uc * sgn), th);
    s.m = (float)fma(a.beta2, (double)s.m, a.one_minus_beta2 * gh);
}

template <int OPT>
__device__ __forceinline__ void apply_elem(const UpdateArgs& a, double h, double uc, float g, ElemState& s)
{
    if constexpr (OPT == ADAGC_OPT_ADAMW) adamw_elem(a, h, uc, g, s);
    else lion_elem(a, h, uc, g, s);
}

template <int OPT>
__device__ __forceinline__ void apply_vec(const UpdateArgs& a, double h, double uc, f32x4 g, f32x4& p, f32x4& m, f32x4& v)
{
    ElemState s;
    s = {p.x, m.x, v.x}; apply_elem<OPT>(a, h, uc, g.x, s); p.x = s.p; m.x = s.m; v.x = s.v;
    s = {p.y, m.y, v.y}; apply_elem<OPT>(a, h, uc, g.y, s); p.y = s.p; m.y = s.m; v.y = s.v;
    s = {p.z, m.z, v.z}; apply_elem<OPT>(a, h, uc, g.z, s); p.z = s.p; m.z = s.m; v.z = s.v;
    s = {p.w, m.w, v.w}; apply_elem<OPT>(a, h, uc, g.w, s); p.w = s.p; m.w = s.m; v.w = s.v;
}

// Telemetry: per-lane fp64 sums of m^2, v^2 and (theta_new - theta_old)^2 over the lane's elements,
// in element order; they become one slot per chunk and per quantity, reduced per tensor afterwards.
template <bool HAS_V>
__device__ __forceinline__ void tele_elem(double (&acc)[3], float p_old, float p_new, float m, float v)
{
    const double dm = (double)m;
    acc[0] = fma(dm, dm, acc[0]);
    if constexpr (HAS_V) {
        const double dv = (double)v;
        acc[1] = fma(dv, dv, acc[1]);
    }
    const double du = (double)p_new - (double)p_old;
    acc[2] = fma(du, du, acc[2]);
}

template <bool HAS_V>
__device__ __forceinline__ void tele_vec(double (&acc)[3], f32x4 p_old, f32x4 p_new, f32x4 m, f32x4 v)
{
    tele_elem<HAS_V>(acc, p_old.x, p_new.x, m.x, v.x);
    tele_elem<HAS_V>(acc, p_old.y, p_new.y, m.y, v.y);
    tele_elem<HAS_V>(acc, p_old.z, p_new.z, m.z, v.z);
    tele_elem<HAS_V>(acc, p_old.w, p_new.w, m.w, v.w);
}

// A tile is U*kBlock consecutive 128-bit vectors (U*1024 elements) of one chunk, handled with U vectors per
// lane and per array in flight; a chunk has kVecPerLane/U tiles.  A workgroup's work item is 1/items_per_chunk
// of a chunk: a run of consecutive tiles (the whole chunk when items_per_chunk is 1).  Small items shorten
// the tail of the launch and give short lists more workgroups; whole chunks cost the fewest dispatches.
// Workgroups are dealt to the XCDs in turn (workgroup b to XCD b mod 8), so items are numbered such that
// eight consecutive workgroups work on eight consecutive positions of the visiting order (one from each of
// its parts) and the items of one chunk all go to the same XCD:
//   item T  ->  position 8*(T / (8*I)) + T % 8,  item (T / 8) % I of that chunk      (I = items_per_chunk, a power of two).
// The items of short chunks follow, from a table of their own.  Tiny chunks, last, go four to a workgroup (the direction's norms
// take them one by one).

struct WorkItem {
    WorkRef chunk;
    int     part;     // which item of the chunk
};

__device__ __forceinline__ uint64_t long_items(const DeviceTables& t, uint32_t log2_items)
{
    return (((uint64_t)t.n_long + 7u) & ~(uint64_t)7u) << log2_items;
}

// Item number `item` of the long and short chunks.  False: this number is only there to fill a group of eight.
__device__ __forceinline__ bool work_item(const DeviceTables& t, uint64_t item, uint32_t log2_items, WorkItem& w)
{
    const uint64_t in_long = long_items(t, log2_items);
    if (item < in_long) {
        const uint32_t k = (uint32_t)(item >> (3 + log2_items)) * 8u + ((uint32_t)item & 7u);
        if (k >= t.n_long) return false;
        w.part = (int)(((uint32_t)item >> 3) & ((1u << log2_items) - 1u));
        w.chunk = load_work(t.work, k);
    } else {
        w.chunk = load_work(t.items, (uint32_t)(item - in_long));
        w.part = (int)(w.chunk.len >> kPartShift);
        w.chunk.len &= (1u << kPartShift) - 1u;
    }
    return true;
}

// The per-tensor rule inside the update kernel (FusedRule); all 64 lanes.  A tensor has at most 64 partial sums: one to a
// lane, the other lanes' and waves' shares of the rules kernel's order are zeros there too, so the sum is the same bit for bit.
// The lane with the tensor's first element stores the results (`stores`).  What it needs is loaded before the elements, and the rule
// evaluated while they are on their way.
struct RuleInputs {
    double partial;
    float  gamma;
};
__device__ __forceinline__ RuleInputs load_rule_inputs(const DeviceTables& t, uint32_t tensor, const TensorArgs& ta)
{
    const uint32_t lane = threadIdx.x & 63u;
    RuleInputs in;
    in.partial = lane < ta.chunk_count ? t.partials[ta.chunk_begin + lane] : 0.0;
    in.gamma = uniform_load(t.ema_before + tensor);
    return in;
}
__device__ __forceinline__ double rule_in_update(const DeviceTables& t, const FusedRule& rule, uint32_t tensor, const RuleInputs& in,
                                                 bool stores)
{
    const double s = wave_sum_f64(in.partial);
    const TensorRule o = adagc_rule(rule.r, s, (double)in.gamma);
    if (stores) store_rule(t, rule.ema, tensor, s, o);
    return o.h;
}

// A chunk's sum of squares by a single wave, in the norm kernel's order: four lanes' shares one after another.
template <bool BF16, int UNROLL>
__device__ __forceinline__ double chunk_sumsq_by_wave(const TensorArgs& ta, uint32_t index, int lane)
{
    const int64_t first = (int64_t)index * kChunkElems, rest = ta.numel - first;
    const int len = rest < kChunkElems ? (int)rest : kChunkElems;
    const gcbytes g = grad_at<BF16>(ta.grad, first);
    if (chunk_kind(len, default_items(UNROLL), UNROLL, 1) == kTinyChunk) return tiny_chunk_sumsq<BF16>(g, len, ta.vec_ok != 0, lane);
    double total = wave_sum_f64(chunk_sumsq_share<BF16, false>(g, len, ta.vec_ok != 0, lane));
#pragma unroll 1
    for (int w = 1; w < kWavesPerBlock; ++w) total += wave_sum_f64(chunk_sumsq_share<BF16, false>(g, len, ta.vec_ok != 0, w * 64 + lane));
    return total;
}

// The rule of a single launch (Exchange), by one wave that has the sum of its chunk: `own`.  publishes: this wave is the one of the
// chunk's that tells it to the others; the one of the tensor's first chunk tells gamma as well, before it may store the new one (`stores`).
// At most 64 chunks, a lane for each.
struct OneLaunchInputs {
    float    gamma;
    uint32_t before;         // (lane 0) launches of this wave so far
};
__device__ __forceinline__ OneLaunchInputs load_one_launch_inputs(const FusedRule& rule, const Exchange& x, uint32_t tensor, bool alone, uint32_t wave)
{
    OneLaunchInputs in{load_shared(rule.ema + tensor), 0u};
    if (!alone && x.launches && (threadIdx.x & 63u) == 0)
        in.before = __hip_atomic_fetch_add(x.launches + wave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return in;
}

template <bool BF16, int UNROLL>
__device__ __forceinline__ double rule_in_one_launch(const DeviceTables& t, const FusedRule& rule, const Exchange& x, const WorkRef& c,
                                                     const TensorArgs& ta, const OneLaunchInputs& in, double own, bool alone, bool publishes)
{
    const uint32_t lane = threadIdx.x & 63u;
    float gamma = in.gamma;
    double mine = lane == c.index ? own : 0.0;
    if (!alone) {
        const uint32_t launch = 1u + (uint32_t)__builtin_amdgcn_readfirstlane((int)in.before);
        asm volatile("" : "+v"(gamma) : : "memory");       // it is here before the first look
        const uint64_t number = (uint64_t)launch << 32;
        uint64_t* const sums = x.words + 2 * (size_t)ta.chunk_begin;
        uint64_t* const gammas = x.words + 2 * (size_t)t.n_chunks;
        if (publishes && lane == 0) {
            store_shared(sums + 2 * c.index, number | (uint32_t)__double2loint(own));
            store_shared(sums + 2 * c.index + 1, number | (uint32_t)__double2hiint(own));
            if (c.index == 0) store_shared(gammas + c.tensor, number | __float_as_uint(gamma));
        }
        bool missing = lane < ta.chunk_count && lane != c.index, gamma_missing = !(publishes && c.index == 0);
        for (uint32_t look = 0;; ++look) {
            const uint32_t at = lane < ta.chunk_count ? lane : 0;
            const uint64_t lo = load_shared(sums + 2 * at), hi = load_shared(sums + 2 * at + 1), g = load_shared(gammas + c.tensor);
            if (missing && (lo >> 32) == launch && (hi >> 32) == launch) {
                mine = __hiloint2double((int)(uint32_t)hi, (int)(uint32_t)lo);
                missing = false;
            }
            if (gamma_missing && (g >> 32) == launch) {
                gamma = __uint_as_float((uint32_t)g);
                gamma_missing = false;
            }
            // (a gamma that has not been told has not been replaced either: what was read above stands)
            if (!__any(missing || gamma_missing) || look >= x.polls) break;
        }
        for (uint64_t left = __ballot(missing); left; left &= left - 1) {
            const uint32_t k = (uint32_t)__builtin_ctzll(left);
            const double s = chunk_sumsq_by_wave<BF16, UNROLL>(ta, k, (int)lane);
            if (lane == k) mine = s;
        }
        // what this wave has told is there for all before the new gamma can be
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (0xF << 8));
        asm volatile("" ::: "memory");
    }
    const double s = wave_sum_f64(mine);
    const TensorRule o = adagc_rule(rule.r, s, (double)gamma);
    if (publishes && c.index == 0 && lane == 0) store_rule(t, rule.ema, c.tensor, s, o);
    return o.h;
}

// All loads of this wave are there before anything else is done.  With seven arrays and a copy to write, stores that start
// while the item's last loads are still on their way cost a little more in read/write turnaround than they gain.  AdamW with the
// copy, without / with the wait: GPT-2-small shapes 686 / 679 us per step, 133 M parameters with bf16 gradients 639 / 635 (664 /
// 660 and 890 / 876 through other entry points), 1.9 B 10.89 / 10.76 ms; 1500 ragged tensors 1.96 both; 5000 small ones lose
// by it, 109 / 113 us.  Without the copy the two are within 1 % on large lists and small ones lose (103 / 106 us); Lion 6.65 /
// 6.71 ms.
__device__ __forceinline__ void wait_for_loads()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (0xF << 8));          // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
}

// Waves per SIMD that the update kernel may have in flight.  With 4 vectors of each array one wave holds 16 loads of 1 KiB, so two are
// enough to cover the latency, and more only open more DRAM rows at once: AdamW on GPT-2-small shapes 657 us per step with 2, 667 with
// 3, 670 with 4 (Llama-3-8B shapes 10.75, 10.90, 10.87 ms for 4 layers).  With 2 vectors AdamW has 4: 5000 small tensors 94 us with 4,
// 98 with 3; GPT-2-small 616 - 630, 622; 133 M parameters with bf16 gradients and copies 630, 640 (ragged tensors end to end 2085,
// 2035).  Lion has fewer arrays in flight and wants 3: GPT-2-small shapes 476 us with 2, 448 with 3, 448 with 4; 1500 ragged tensors
// 1518, 1450, 1495; Llama-3-8B shapes with bf16 gradients and copies 7.10, 6.65, 6.97 ms (5000 small tensors 88, 77, 72 us).  A single
// launch, of a round of workgroups at most, has the registers of two.
template <int OPT, int U>
constexpr int kUpdateWaves = OPT == ADAGC_OPT_ADAMW ? (U == 4 ? 2 : 4) : 3;

// Whether the per-tensor rule is evaluated here: known where the launch is one of the library's own choice, else asked.
// kRuleOne: and the chunks' sums of squares as well (Exchange).
enum RuleHere { kRuleNo, kRuleYes, kRuleAsk, kRuleOne };

template <int OPT, bool BF16G, bool COPY, int U, bool NT, bool TELE, bool LINES, RuleHere RULE>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(RULE == kRuleOne ? 2 : kUpdateWaves<OPT, U>, RULE == kRuleOne ? 2 : kUpdateWaves<OPT, U>)))
void update_kernel(DeviceTables t, UpdateArgs a, uint32_t log2_items, const StepScalars* device_scalars, FusedRule rule, Exchange exchange)
{
    static_assert(kVecPerLane % U == 0, "a chunk is a whole number of tiles");
    if (device_scalars) {                      // adagc_step_graph: this step's scalars live in device memory
        if (device_scalars->status != 0) return;
        a = device_scalars->u;
    }
    constexpr bool NTL = NT, NTS = NT;    // non-temporal loads and stores
    constexpr bool kHasV = (OPT == ADAGC_OPT_ADAMW);
    constexpr int kTiles = kVecPerLane / U;
    const int tid = threadIdx.x;
    __shared__ double tele_sums[3][kWavesPerBlock];
    __shared__ double one_sums[kWavesPerBlock + 1];        // a single launch: the waves' sums, then the coefficient

    // Tiles first_tile .. first_tile + n_tiles - 1 of a chunk, by LANES lanes (a workgroup, or a wave of it).
    auto update_tiles = [&](auto LANES, const WorkRef& c, int first_tile, int n_tiles, int lane, double (&tele)[3])
                            __attribute__((always_inline)) {
        constexpr int kLanes = decltype(LANES)::value;
        constexpr int kTileVecs = U * kLanes, kTileElems = kTileVecs * 4;
        const uint32_t tensor = c.tensor;
        const int len = (int)c.len;
        const int64_t first = first_element(c);
        const TensorArgs ta = load_tensor(t.targs, tensor);
        // the tensor's coefficient as computed, in double
        double h = 1.0;
        RuleInputs rule_inputs{0.0, 0.f};
        if constexpr (RULE == kRuleYes) rule_inputs = load_rule_inputs(t, tensor, ta);
        if constexpr (RULE == kRuleAsk)        // (before the elements: a branch between their loads and their use costs more, where the rule has run)
            h = rule.ema ? rule_in_update(t, rule, tensor, load_rule_inputs(t, tensor, ta), c.index == 0 && first_tile == 0 && lane == 0)
                         : uniform_load(t.coef64 + tensor);
        if constexpr (RULE == kRuleNo) h = uniform_load(t.coef64 + tensor);
        auto evaluate_rule = [&]() __attribute__((always_inline)) {
            if constexpr (RULE == kRuleOne) {
                const gcbytes chunk = grad_at<BF16G>(ta.grad, first);
                const bool alone = ta.chunk_count == 1 && len <= kTiles / default_items(U) * U * kBlock * 4;
                const uint32_t wave = blockIdx.x * kWavesPerBlock + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
                OneLaunchInputs in{};
                if (lane < 64) in = load_one_launch_inputs(rule, exchange, tensor, alone, wave);
                if constexpr (kLanes == 64) {
                    const double own = tiny_chunk_sumsq<BF16G>(chunk, len, ta.vec_ok != 0, lane);
                    h = rule_in_one_launch<BF16G, U>(t, rule, exchange, c, ta, in, own, alone, true);
                } else {
                    const double share = wave_sum_f64(chunk_sumsq_share<BF16G, false>(chunk, len, ta.vec_ok != 0, lane));
                    if ((lane & 63) == 0) one_sums[lane >> 6] = share;
                    __syncthreads();
                    if (lane < 64) {
                        double own = one_sums[0];
#pragma unroll
                        for (int w = 1; w < kWavesPerBlock; ++w) own += one_sums[w];
                        const double coef = rule_in_one_launch<BF16G, U>(t, rule, exchange, c, ta, in, own, alone, first_tile == 0);
                        if (lane == 0) one_sums[kWavesPerBlock] = coef;
                    }
                    __syncthreads();
                    h = one_sums[kWavesPerBlock];
                }
            }
            if constexpr (RULE == kRuleYes) h = rule_in_update(t, rule, tensor, rule_inputs, c.index == 0 && first_tile == 0 && lane == 0);
        };
        const double uc = a.update_clip ? uniform_load(t.ucoef64 + tensor) : 1.0;   // update clipping: scales the direction
        const gcbytes g = grad_at<BF16G>(ta.grad, first);
        const gfloat p = (gfloat)ta.param + first;
        const gfloat m = (gfloat)ta.exp_avg + first;
        const gfloat v = kHasV ? (gfloat)ta.exp_avg_sq + first : nullptr;
        const gu16 pc = COPY ? (gu16)ta.param_copy + first : nullptr;

#pragma unroll 1
        for (int tt = 0; tt < n_tiles; ++tt) {
            const int sub = first_tile + tt;
            const int e0 = sub * kTileElems;                                   // the tile's elements inside the chunk:
            const int e1 = len < e0 + kTileElems ? len : e0 + kTileElems; // [e0, e1), empty past a ragged end
            if (e0 >= e1) break;
            if (ta.vec_ok) {
                // LINES: tiles start on a line.  A wave's access to 16 bytes per lane that does not touches nine lines instead of eight,
                // two of them in part, and of a line written in part the memory writes what is there anew.  So where the arrays
                // agree on their place in a line, every tile of the tensor is taken `shift` elements earlier: a chunk's first tile has
                // the end of the chunk before it, the tensor's last tile what is left, one by one.  Tensors laid end to end (1500 of
                // up to 4 M elements): 2290 us per step without, 2062 with.  (Not with telemetry: its partial sums
                // would have the elements in another order than on tensors that lie apart.)  Lists that lie on lines, small lists and
                // small launches (walk_lines.h) have a kernel without the shift: 5000 small tensors 102 us there, 112 here.
                const int shift = LINES ? (int)ta.line_offset : 0;
                const bool starts = LINES && c.index == 0, ends = !LINES || c.index + 1 == ta.chunk_count;
                const auto p4 = (ADAGC_GLOBAL f32x4_any*)(p - shift);
                const auto m4 = (ADAGC_GLOBAL f32x4_any*)(m - shift);
                const auto v4 = (ADAGC_GLOBAL f32x4_any*)(kHasV ? v - shift : nullptr);
                const auto c4 = (ADAGC_GLOBAL u32x2_any*)(COPY ? pc - shift : nullptr);
                const gcbytes g4 = g - shift * (BF16G ? 2 : 4);
                const int v0 = sub * kTileVecs;

                // Whole tiles and ragged ends alike: all loads before the first store (in a loop over the vectors of a
                // ragged end they would wait for the stores of the round before).  Lanes outside the whole vectors
                // vmin .. nvec - 1 load the nearest one and store nothing; up to three single elements come with the tile that
                // starts the tensor, up to three (and the 31 that no tile has) with the one that ends it.
                const int vmin = starts ? (shift + 3) >> 2 : 0;
                const int nvec = ends ? (len + shift) >> 2 : kChunkElems / 4;
                int j = (nvec << 2) + lane;
                bool any = v0 < nvec, single = e1 == len && j < len;
                if constexpr (LINES) {
                    const int vend = nvec < v0 + kTileVecs ? nvec : v0 + kTileVecs;
                    any = (v0 > vmin ? v0 : vmin) < vend;
                    const int before = starts && sub == 0 ? 4 * vmin - shift : 0, n_head = before < len ? before : len;
                    const int tail = starts && vend <= vmin ? n_head : 4 * vend - shift;
                    const int n_tail = ends && e1 == len ? len - tail : 0;
                    j = lane < n_head ? lane : tail + lane - n_head;
                    single = lane < n_head + n_tail;
                }
                ElemState s = {0.f, 0.f, 0.f};
                float g1 = 0.f;
                if (single) {
                    s = {p[j], m[j], kHasV ? v[j] : 0.f};
                    g1 = load_grad1<BF16G>(g, j);
                }
                if (any) {
                    f32x4 gg[U], pp[U], mm[U], vv[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int want = v0 + u * kLanes + lane, most = want < nvec ? want : nvec - 1, idx = LINES && most < vmin ? vmin : most;
                        gg[u] = load_grad4<BF16G, NTL>(g4, idx);
                        pp[u] = ld<NTL>(p4 + idx);
                        mm[u] = ld<NTL>(m4 + idx);
                        if constexpr (kHasV) vv[u] = ld<NTL>(v4 + idx);
                        else vv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                    if (tt == 0) evaluate_rule();
                    if constexpr (kHasV && COPY) wait_for_loads();
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int idx = v0 + u * kLanes + lane;
                        if (idx >= nvec) break;
                        if (LINES && idx < vmin) continue;
                        const f32x4 p_old = pp[u];
                        apply_vec<OPT>(a, h, uc, gg[u], pp[u], mm[u], vv[u]);
                        if constexpr (TELE) tele_vec<kHasV>(tele, p_old, pp[u], mm[u], vv[u]);
                        st<NTS>(p4 + idx, pp[u]);
                        st<NTS>(m4 + idx, mm[u]);
                        if constexpr (kHasV) st<NTS>(v4 + idx, vv[u]);
                        if constexpr (COPY) st<NTS>(c4 + idx, pack_bf16x4(pp[u]));
                    }
                } else if (tt == 0) {
                    evaluate_rule();
                }
                if (single) {
                    const float p_old = s.p;
                    apply_elem<OPT>(a, h, uc, g1, s);
                    if constexpr (TELE) tele_elem<kHasV>(tele, p_old, s.p, s.m, s.v);
                    p[j] = s.p;
                    m[j] = s.m;
                    if constexpr (kHasV) v[j] = s.v;
                    if constexpr (COPY) pc[j] = (uint16_t)float_to_bf16_bits(s.p);
                }
            } else {
                if (tt == 0) evaluate_rule();
                for (int j = e0 + lane; j < e1; j += kLanes) {
                    ElemState s = {p[j], m[j], kHasV ? v[j] : 0.f};
                    const float p_old = s.p;
                    apply_elem<OPT>(a, h, uc, load_grad1<BF16G>(g, j), s);
                    if constexpr (TELE) tele_elem<kHasV>(tele, p_old, s.p, s.m, s.v);
                    p[j] = s.p;
                    m[j] = s.m;
                    if constexpr (kHasV) v[j] = s.v;
                    if constexpr (COPY) pc[j] = (uint16_t)float_to_bf16_bits(s.p);
                }
            }
        }

    };

    const int tiles_per_item = kTiles >> log2_items;
    const uint32_t n_wide = t.n_chunks - t.n_tiny;
    const uint64_t n_wide_items = long_items(t, log2_items) + t.n_short, n_items = n_wide_items + (t.n_tiny + 3u) / 4u;
    for (uint64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        double tele[3] = {0.0, 0.0, 0.0};
        if (item >= n_wide_items) {            // four tiny chunks, one to a wave
            const uint32_t at = n_wide + (uint32_t)(item - n_wide_items) * 4u + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
            if (at < t.n_chunks) {
                const WorkRef c = load_work(t.work, at);
                update_tiles(std::integral_constant<int, 64>{}, c, 0, 1, tid & 63, tele);
                if constexpr (TELE) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const double part = wave_sum_f64(tele[q]);
                        if ((tid & 63) == 0) t.tele_partials[((size_t)q * t.n_chunks + c.slot) << log2_items] = part;
                    }
                }
            }
            continue;
        }
        WorkItem w;
        if (!work_item(t, item, log2_items, w)) continue;
        update_tiles(std::integral_constant<int, kBlock>{}, w.chunk, w.part * tiles_per_item, tiles_per_item, tid, tele);

        if constexpr (TELE) {
            // every item writes its slots; those that a chunk of one item has no item for stay zero from the start
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const double part = wave_sum_f64(tele[q]);
                if ((tid & 63) == 0) tele_sums[q][tid >> 6] = part;
            }
            __syncthreads();
            if (tid < 3) {
                double b = tele_sums[tid][0];
#pragma unroll
                for (int k = 1; k < kWavesPerBlock; ++k) b += tele_sums[tid][k];
                t.tele_partials[(((size_t)tid * t.n_chunks + w.chunk.slot) << log2_items) + w.part] = b;
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Update clipping (AGC and Clippy rows of Table 2).  The coefficient of a tensor's update needs the norms
// of theta and of the whole tensor's direction Delta, so the direction is evaluated twice: here for its
// norms (nothing is written but two partial results per work item), then by update_kernel, which scales it.
// Work items are those of update_kernel, or several of them (log2_stats_items).  LINF selects maxima of |.| (Clippy) instead of sums of
// squares (AGC).

// All 64 lanes must be active.  Returns the same value in every lane.  Maxima are exact in any order.
__device__ __forceinline__ double wave_max_f64(double x)
{
    x = fmax(x, dpp_mov<0x128>(x));  // row_ror:8
    x = fmax(x, dpp_mov<0x124>(x));  // row_ror:4
    x = fmax(x, dpp_mov<0x122>(x));  // row_ror:2
    x = fmax(x, dpp_mov<0x121>(x));  // row_ror:1
    return fmax(fmax(readlane_f64(x, 0), readlane_f64(x, 16)), fmax(readlane_f64(x, 32), readlane_f64(x, 48)));
}

// The direction of one element for the unclipped gradient: AdamW m_hat/(sqrt(v_hat)+eps) from this step's
// moments, Lion the sign of the interpolation.
template <int OPT>
__device__ __forceinline__ double direction_elem(const UpdateArgs& a, float g, float m_prev, float v_prev)
{
    const double gd = (double)g;
    if constexpr (OPT == ADAGC_OPT_ADAMW) {
        const double m = fma(a.beta1, (double)m_prev, a.one_minus_beta1 * gd);
        const double v = fma(a.beta2, (double)v_prev, a.one_minus_beta2 * gd * gd);
        return (m * a.inv_bias1) / (sqrt(v * a.inv_bias2) + a.eps);
    } else {
        return lion_sign(a, gd, m_prev);
    }
}

template <bool LINF>
__device__ __forceinline__ void stat_acc(double (&acc)[2], float theta, double delta)
{
    const double th = (double)theta;
    if constexpr (LINF) {
        acc[0] = fmax(acc[0], fabs(th));       // a NaN never becomes the maximum
        acc[1] = fmax(acc[1], fabs(delta));
    } else {
        acc[0] = fma(th, th, acc[0]);
        acc[1] = fma(delta, delta, acc[1]);
    }
}

// Vectors per lane and array in flight.  AdamW: 4 whatever the update kernel has; with 2, and 2048 elements at a time, 133 M
// parameters under AGC take 932 us per step, so 919.
template <int OPT>
constexpr int kStatsUnroll = OPT == ADAGC_OPT_ADAMW ? 4 : 2;

// Items of a long chunk, where the update kernel has 1 << log2_items: none smaller than a tile.
template <int OPT>
__host__ __device__ constexpr uint32_t log2_stats_items(uint32_t log2_items)
{
    constexpr uint32_t kMost = kVecPerLane / kStatsUnroll<OPT>;
    static_assert((kMost & (kMost - 1)) == 0, "a power of two");
    return (1u << log2_items) < kMost ? log2_items : (uint32_t)__builtin_ctz(kMost);
}

template <int OPT, bool BF16G, bool LINF, bool NT>
__global__ __launch_bounds__(kBlock) void direction_stats_kernel(DeviceTables t, UpdateArgs a, uint32_t log2_items)
{
    constexpr int U = kStatsUnroll<OPT>;
    constexpr bool kHasV = (OPT == ADAGC_OPT_ADAMW);
    constexpr int kTileVecs = U * kBlock;
    constexpr int kTileElems = kTileVecs * 4;
    const int tid = threadIdx.x;
    __shared__ double wave_part[2][kWavesPerBlock];

    // a long chunk's items are taken as many at a time as make a tile, for the slot of the first of them
    const uint32_t log2_long = log2_stats_items<OPT>(log2_items);
    const uint64_t in_long = long_items(t, log2_long), n_wide_items = in_long + t.n_short, n_items = n_wide_items + t.n_tiny;
    for (uint64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        WorkItem w;
        if (item >= n_wide_items) w = {load_work(t.work, t.n_chunks - t.n_tiny + (uint32_t)(item - n_wide_items)), 0};
        else if (!work_item(t, item, log2_long, w)) continue;
        if (item < in_long) w.part <<= log2_items - log2_long;
        const int item_elems = kChunkElems >> (item < in_long ? log2_long : log2_items);         // may be less than a tile: the caller chooses
        const int len = (int)w.chunk.len;
        const int64_t first = first_element(w.chunk);
        const TensorArgs ta = load_tensor(t.targs, w.chunk.tensor);
        const gcbytes g = grad_at<BF16G>(ta.grad, first);
        const gcfloat p = (gcfloat)ta.param + first;
        const gcfloat m = (gcfloat)ta.exp_avg + first;
        const gcfloat v = kHasV ? (gcfloat)ta.exp_avg_sq + first : nullptr;
        double acc[2] = {0.0, 0.0};

        const int item_begin = w.part * (kChunkElems >> log2_items);
        const int item_end = len < item_begin + item_elems ? len : item_begin + item_elems;
#pragma unroll 1
        for (int e0 = item_begin; e0 < item_end; e0 += kTileElems) {
            const int e1 = item_end < e0 + kTileElems ? item_end : e0 + kTileElems;
            if (ta.vec_ok) {
                const auto p4 = (const ADAGC_GLOBAL f32x4_any*)p;
                const auto m4 = (const ADAGC_GLOBAL f32x4_any*)m;
                const auto v4 = (const ADAGC_GLOBAL f32x4_any*)v;
                const int v0 = e0 >> 2, vend = e1 >> 2;
                if (e1 - e0 == kTileElems) {
                    f32x4 gg[U], pp[U], mm[U], vv[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int idx = v0 + u * kBlock + tid;
                        gg[u] = load_grad4<BF16G, NT>(g, idx);
                        pp[u] = ld<NT>(p4 + idx);
                        mm[u] = ld<NT>(m4 + idx);
                        if constexpr (kHasV) vv[u] = ld<NT>(v4 + idx);
                        else vv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        stat_acc<LINF>(acc, pp[u].x, direction_elem<OPT>(a, gg[u].x, mm[u].x, vv[u].x));
                        stat_acc<LINF>(acc, pp[u].y, direction_elem<OPT>(a, gg[u].y, mm[u].y, vv[u].y));
                        stat_acc<LINF>(acc, pp[u].z, direction_elem<OPT>(a, gg[u].z, mm[u].z, vv[u].z));
                        stat_acc<LINF>(acc, pp[u].w, direction_elem<OPT>(a, gg[u].w, mm[u].w, vv[u].w));
                    }
                } else {
                    for (int idx = v0 + tid; idx < vend; idx += kBlock) {
                        const f32x4 gg = load_grad4<BF16G, NT>(g, idx);
                        const f32x4 pp = ld<NT>(p4 + idx);
                        const f32x4 mm = ld<NT>(m4 + idx);
                        f32x4 vv = f32x4{0.f, 0.f, 0.f, 0.f};
                        if constexpr (kHasV) vv = ld<NT>(v4 + idx);
                        stat_acc<LINF>(acc, pp.x, direction_elem<OPT>(a, gg.x, mm.x, vv.x));
                        stat_acc<LINF>(acc, pp.y, direction_elem<OPT>(a, gg.y, mm.y, vv.y));
                        stat_acc<LINF>(acc, pp.z, direction_elem<OPT>(a, gg.z, mm.z, vv.z));
                        stat_acc<LINF>(acc, pp.w, direction_elem<OPT>(a, gg.w, mm.w, vv.w));
                    }
                    const int j = (vend << 2) + tid;            // up to three single elements at the ragged end
                    if (j < e1)
                        stat_acc<LINF>(acc, p[j], direction_elem<OPT>(a, load_grad1<BF16G>(g, j), m[j], kHasV ? v[j] : 0.f));
                }
            } else {
                for (int j = e0 + tid; j < e1; j += kBlock)
                    stat_acc<LINF>(acc, p[j], direction_elem<OPT>(a, load_grad1<BF16G>(g, j), m[j], kHasV ? v[j] : 0.f));
            }
        }

        // every item writes its two slots, a long chunk's those of the first of the update kernel's items that it covers; the others are
        // never written and zero since the context's creation, which adds nothing to either norm
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double part = LINF ? wave_max_f64(acc[q]) : wave_sum_f64(acc[q]);
            if ((tid & 63) == 0) wave_part[q][tid >> 6] = part;
        }
        __syncthreads();
        if (tid < 2) {
            double b = wave_part[tid][0];
#pragma unroll
            for (int v = 1; v < kWavesPerBlock; ++v) b = LINF ? fmax(b, wave_part[tid][v]) : b + wave_part[tid][v];
            t.ustat_partials[(((size_t)tid * t.n_chunks + w.chunk.slot) << log2_items) + w.part] = b;
        }
        __syncthreads();
    }
}

// The maximum of a tensor's slots (any order gives the same value).
__device__ __forceinline__ double tensor_slot_max(const DeviceTables& t, const double* slots, uint32_t i, double* wave_part,
                                                  uint32_t slots_per_chunk)
{
    const uint32_t count = t.targs[i].chunk_count * slots_per_chunk;
    const double* p = slots + (size_t)t.targs[i].chunk_begin * slots_per_chunk;
    // eight loads at a time: one by one an embedding of 39 M elements, with eight slots a chunk, takes 20 us
    constexpr int kFlight = 8;
    double a0 = 0.0;
    uint32_t k = threadIdx.x;
    for (; k + (kFlight - 1) * kBlock < count; k += kFlight * kBlock) {
        double x[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) x[u] = p[k + u * kBlock];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) a0 = fmax(a0, x[u]);
    }
    for (; k < count; k += kBlock) a0 = fmax(a0, p[k]);
    const double s = wave_max_f64(a0);
    if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = s;
    __syncthreads();
    double total = wave_part[0];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) total = fmax(total, wave_part[w]);
    return total;
}

// One workgroup per tensor: the two norms from the item slots, then Table 2's AGC or Clippy coefficient.
// The gradient's own coefficient is 1 in these modes.  Reported to the caller: the direction's norm,
// the update coefficient, and whether it is below 1.
__global__ __launch_bounds__(kBlock) void finalize_update_clip_kernel(DeviceTables t, RuleArgs r, uint32_t items_per_chunk)
{
    __shared__ double wave_part[kWavesPerBlock];
    const uint32_t i = blockIdx.x;
    const bool linf = r.mode == ADAGC_MODE_CLIPPY;
    double stat[2];
    for (int q = 0; q < 2; ++q) {
        const double* slots = t.ustat_partials + (size_t)q * t.n_chunks * items_per_chunk;
        stat[q] = linf ? tensor_slot_max(t, slots, i, wave_part, items_per_chunk)
                       : tensor_slot_sum(t, slots, i, wave_part, items_per_chunk);
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    double ratio, delta_norm;
    if (linf) {
        delta_norm = stat[1];
        ratio = __ddiv_rn(__dadd_rn(__dmul_rn(r.lambda_rel, stat[0]), r.lambda_abs), __dmul_rn(r.lr, delta_norm));
    } else {
        delta_norm = sqrt(stat[1]);
        ratio = __ddiv_rn(__dmul_rn(r.lambda_rel, sqrt(stat[0])), delta_norm);
    }
    const bool active = ratio < 1.0;              // false for NaN (0/0): the update is left alone
    const double c = active ? ratio : 1.0;
    t.norm[i] = (float)delta_norm;
    t.coef[i] = (float)c;
    t.ucoef64[i] = c;
    t.coef64[i] = 1.0;
    t.flag[i] = active ? 1 : 0;
}

// Telemetry: workgroup (i, q) turns tensor i's item slots of quantity q into its norm (same fixed order as K2).
__global__ __launch_bounds__(kBlock) void finalize_telemetry_kernel(DeviceTables t, uint32_t items_per_chunk)
{
    __shared__ double wave_sums[kWavesPerBlock];
    const uint32_t i = blockIdx.x, q = blockIdx.y;
    const double s = tensor_slot_sum(t, t.tele_partials + (size_t)q * t.n_chunks * items_per_chunk, i, wave_sums, items_per_chunk);
    if (threadIdx.x == 0) t.tele_norm[(size_t)q * t.n_tensors + i] = (float)sqrt(s);
}

using UpdateFn = void (*)(DeviceTables, UpdateArgs, uint32_t, const StepScalars*, FusedRule, Exchange);

// Where whole lines ever pay, the launches of the library's own choice (streaming, so many vectors in flight) have kernels with
// them; those of lists that may be small have kernels with and without the rule.
template <int OPT, bool BF16G, bool COPY, int U, RuleHere RULE>
UpdateFn select_update_flags(int nt, int tele, bool lines)
{
    if constexpr (lines_with_unroll(OPT, U) && line_limits(OPT, BF16G, COPY).elems > 0)
        if (lines && nt && !tele) return update_kernel<OPT, BF16G, COPY, U, true, false, true, RULE>;
    if (nt) return tele ? update_kernel<OPT, BF16G, COPY, U, true, true, false, RULE> : update_kernel<OPT, BF16G, COPY, U, true, false, false, RULE>;
    return tele ? update_kernel<OPT, BF16G, COPY, U, false, true, false, kRuleAsk> : update_kernel<OPT, BF16G, COPY, U, false, false, false, kRuleAsk>;
}

template <int OPT, bool BF16G, bool COPY>
UpdateFn select_update_variant(int unroll, int nt, int tele, bool lines, bool rule, bool one)
{
    if (one) return update_kernel<OPT, BF16G, COPY, default_unroll(OPT), true, false, false, kRuleOne>;
    static_assert(default_unroll(OPT) == 2, "the kernels below");
    // (With bf16 gradients and no copy the kernel that asks is the quicker one where the rule has run: 231 M parameters, without / asked: static 1072 /
    // 1050 us per step, recorded 1079 / 1056, GlobalGC-like rules 1046 / 1034, 421 M static 2015 / 1991; with telemetry 1073 / 1085.)
    if constexpr (OPT == ADAGC_OPT_ADAMW)
        if (unroll == 4)
            return rule ? select_update_flags<OPT, BF16G, COPY, 4, kRuleYes>(nt, tele, lines)
                        : select_update_flags<OPT, BF16G, COPY, 4, BF16G && !COPY ? kRuleAsk : kRuleNo>(nt, tele, lines);
    if (unroll == 4) return select_update_flags<OPT, BF16G, COPY, 4, kRuleAsk>(nt, tele, lines);
    if (unroll == 1) return select_update_flags<OPT, BF16G, COPY, 1, kRuleAsk>(nt, tele, lines);
    return rule ? select_update_flags<OPT, BF16G, COPY, 2, kRuleYes>(nt, tele, lines) : select_update_flags<OPT, BF16G, COPY, 2, kRuleNo>(nt, tele, lines);
}

UpdateFn select_update(int optimizer, int grad_bf16, int with_copy, int unroll, int nt, int tele, bool lines, bool rule, bool one)
{
    const int key = (optimizer == ADAGC_OPT_LION ? 4 : 0) | (grad_bf16 ? 2 : 0) | (with_copy ? 1 : 0);
    switch (key) {
    case 0: return select_update_variant<ADAGC_OPT_ADAMW, false, false>(unroll, nt, tele, lines, rule, one);
    case 1: return select_update_variant<ADAGC_OPT_ADAMW, false, true>(unroll, nt, tele, lines, rule, one);
    case 2: return select_update_variant<ADAGC_OPT_ADAMW, true, false>(unroll, nt, tele, lines, rule, one);
    case 3: return select_update_variant<ADAGC_OPT_ADAMW, true, true>(unroll, nt, tele, lines, rule, one);
    case 4: return select_update_variant<ADAGC_OPT_LION, false, false>(unroll, nt, tele, lines, rule, one);
    case 5: return select_update_variant<ADAGC_OPT_LION, false, true>(unroll, nt, tele, lines, rule, one);
    case 6: return select_update_variant<ADAGC_OPT_LION, true, false>(unroll, nt, tele, lines, rule, one);
    default: return select_update_variant<ADAGC_OPT_LION, true, true>(unroll, nt, tele, lines, rule, one);
    }
}

}  // namespace

using NormFn = void (*)(DeviceTables, const adagc_step_params*, int, const float*);

hipError_t launch_sumsq_partials(const DeviceTables& t, int grad_bf16, bool streaming, int grid, hipStream_t stream,
                                 const adagc_step_params* params, int optimizer, const float* ema_to_keep)
{
    const NormFn fn = grad_bf16 ? (streaming ? sumsq_partials_kernel<true, true> : sumsq_partials_kernel<true, false>)
                                : (streaming ? sumsq_partials_kernel<false, true> : sumsq_partials_kernel<false, false>);
    fn<<<dim3(grid), dim3(kBlock), 0, stream>>>(t, params, optimizer, ema_to_keep);
    return hipGetLastError();
}

hipError_t launch_rules(const DeviceTables& t, float* ema, const RuleArgs& r, hipStream_t stream, const adagc_step_params* params,
                        int optimizer)
{
    rules_kernel<<<dim3(t.n_tensors), dim3(kBlock), 0, stream>>>(t, ema, r, params, optimizer);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || t.n_tensors <= kFewTensors || (!params && !model_wide(r))) return e;
    global_rule_kernel<<<dim3(1), dim3(kBlock), 0, stream>>>(t, ema, r, params, optimizer);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint32_t blocks = (t.n_tensors + kBlock - 1) / kBlock;
    finalize_global_kernel<<<dim3(blocks), dim3(kBlock), 0, stream>>>(t, ema, r, params, optimizer);
    return hipGetLastError();
}

hipError_t launch_tensor_rules(const DeviceTables& t, float* ema, const RuleArgs& r, uint32_t first, uint32_t count, hipStream_t stream)
{
    tensor_rules_kernel<<<dim3(count), dim3(kBlock), 0, stream>>>(t, ema, r, first);
    return hipGetLastError();
}

hipError_t launch_tensor_sumsq(const DeviceTables& t, hipStream_t stream)
{
    tensor_sumsq_kernel<<<dim3(t.n_tensors), dim3(kBlock), 0, stream>>>(t);
    return hipGetLastError();
}

using StatsFn = void (*)(DeviceTables, UpdateArgs, uint32_t);

static uint32_t log2_of(int power_of_two) { return (uint32_t)__builtin_ctz((unsigned)power_of_two); }

template <int OPT, bool BF16G>
static StatsFn select_stats_flags(bool linf, int nt)
{
    if (linf) return nt ? direction_stats_kernel<OPT, BF16G, true, true> : direction_stats_kernel<OPT, BF16G, true, false>;
    return nt ? direction_stats_kernel<OPT, BF16G, false, true> : direction_stats_kernel<OPT, BF16G, false, false>;
}

hipError_t launch_update_clip_rule(const DeviceTables& t, const UpdateArgs& u, const RuleArgs& r, int optimizer,
                                   int grad_bf16, int items_per_chunk, int nt, int grid, hipStream_t stream)
{
    const bool linf = r.mode == ADAGC_MODE_CLIPPY;
    const bool lion = optimizer == ADAGC_OPT_LION;
    const StatsFn fn = grad_bf16 ? (lion ? select_stats_flags<ADAGC_OPT_LION, true> : select_stats_flags<ADAGC_OPT_ADAMW, true>)(linf, nt)
                                 : (lion ? select_stats_flags<ADAGC_OPT_LION, false> : select_stats_flags<ADAGC_OPT_ADAMW, false>)(linf, nt);
    const uint32_t log2_items = log2_of(items_per_chunk);
    const uint32_t log2_long = lion ? log2_stats_items<ADAGC_OPT_LION>(log2_items) : log2_stats_items<ADAGC_OPT_ADAMW>(log2_items);
    const int64_t items = ((((int64_t)t.n_long + 7) & ~(int64_t)7) << log2_long) + t.n_short + t.n_tiny;
    fn<<<dim3((uint32_t)(items < grid ? items : grid)), dim3(kBlock), 0, stream>>>(t, u, log2_items);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    finalize_update_clip_kernel<<<dim3(t.n_tensors), dim3(kBlock), 0, stream>>>(t, r, (uint32_t)items_per_chunk);
    return hipGetLastError();
}

hipError_t launch_update(const DeviceTables& t, const UpdateArgs& a, int optimizer, int grad_bf16,
                         int with_copy, int unroll, int items_per_chunk, int nt, int tele, int grid,
                         hipStream_t stream, bool device_scalars, const FusedRule& rule, const Exchange& exchange)
{
    const UpdateFn fn = select_update(optimizer, grad_bf16, with_copy, unroll, nt, tele, t.off_lines != 0, rule.ema != nullptr, exchange.words != nullptr);
    fn<<<dim3(grid), dim3(kBlock), 0, stream>>>(t, a, log2_of(items_per_chunk), device_scalars ? t.scalars : nullptr, rule, exchange);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !tele) return e;
    finalize_telemetry_kernel<<<dim3(t.n_tensors, 3), dim3(kBlock), 0, stream>>>(t, (uint32_t)items_per_chunk);
    return hipGetLastError();
}

}  // namespace adagc
