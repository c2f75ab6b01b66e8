// Elementwise kernels of the Muon step with AdaGC's clipped gradient (Muon is the optimizer the paper pairs
// AdaGC with in "Optimizer Compatibility: Muon and Lion", Sec. 5.4; its rule is the published one, the paper
// prints none):
//
//   muon_momentum_kernel    per chunk:  M <- mu M + h g;  partial sum of squares of U
//                                       (U = h g + mu M in the Nesterov form, U = M otherwise)
//   muon_normalise_kernel   per round:  X0 = bf16(U / (||U||_F + 1e-7)) of every matrix into the zero-padded workspace,
//                                       tall ones transposed
//   muon_apply_kernel       per round:  theta <- theta - lr (wd theta + scale O) of every matrix, optional bf16 copy
//
// A round, all batches that are in the workspace together, is one launch of each over all of its matrices: a matrix of a few hundred
// rows is read in two microseconds, less than a launch takes.  48 hidden matrices of GPT-2-small (85 M parameters, bf16 gradients, three
// batches): normalise 119 us (48 x 7.7 with a launch per matrix; 8 B per parameter), apply 177 us (48 x 6.0; 12 B).  872 M
// parameters at Llama-3-8B shapes, fp32 gradients: normalise 1.65 ms (10 B; with X and its transpose to write 1.94), apply 1.55 ms
// (10 B).
//
// The clip coefficient h of every tensor comes from the same norm and rule kernels as for AdamW and Lion
// (kernels.hip); the Newton-Schulz products run in muon_gemm.hip.  Arithmetic is double with one rounding per
// stored value, as in the other update kernels; reductions are in fixed order.

#include "adagc_device.h"
#include "muon_internal.h"

namespace adagc {
namespace {

// M' and U of one element.  The momentum is stored as fp32; U uses the stored value.
__device__ __forceinline__ double momentum_elem(double h, double mu, int nesterov, float g, float m_prev, float* m_new)
{
    const double gh = h * (double)g;
    const float m = (float)(mu * (double)m_prev + gh);
    *m_new = m;
    return nesterov ? gh + mu * (double)m : (double)m;
}

__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);    // a fixed butterfly: same value in every lane
    return x;
}

// One workgroup per chunk (positions b, b+grid, ... of the list): momentum update and the chunk's sum of U^2.
// Tensors whose pointers allow it are walked in 128-bit vectors (4 elements per lane and access, streaming loads
// and stores: every element is touched once per kernel); the others, and the last len mod 4 elements, one by one.
template <bool BF16>
__global__ __launch_bounds__(kBlock) void muon_momentum_kernel(DeviceTables t, double mu, int nesterov)
{
    __shared__ double wave_sums[kWavesPerBlock];
    const int tid = threadIdx.x;
    for (uint32_t k = blockIdx.x; k < t.n_chunks; k += gridDim.x) {
        const WorkRef ck = load_work(t.work, k);                // the visiting order of the norm kernel (XCD-aware)
        const TensorArgs ta = load_tensor(t.targs, ck.tensor);
        const int len = (int)ck.len;
        const double h = uniform_load(t.coef64 + ck.tensor);
        const gcbytes g0 = grad_at<BF16>(ta.grad, first_element(ck));
        const gfloat m = (gfloat)ta.exp_avg + first_element(ck);
        double acc = 0.0;
        int done = 0;
        if (ta.vec_ok) {
            const int groups = len / 4;
            const auto m4 = (ADAGC_GLOBAL f32x4_any*)m;
            auto update4 = [&](int j, const f32x4 g, const f32x4 mp) {
                f32x4 mn;
                float e;
                double u = momentum_elem(h, mu, nesterov, g.x, mp.x, &e); mn.x = e; acc = fma(u, u, acc);
                u = momentum_elem(h, mu, nesterov, g.y, mp.y, &e); mn.y = e; acc = fma(u, u, acc);
                u = momentum_elem(h, mu, nesterov, g.z, mp.z, &e); mn.z = e; acc = fma(u, u, acc);
                u = momentum_elem(h, mu, nesterov, g.w, mp.w, &e); mn.w = e; acc = fma(u, u, acc);
                st<true>(m4 + j, mn);
            };
            if (len == kChunkElems) {
                // a full chunk is 16 vectors per lane: 8 of each array in flight at a time
                constexpr int kPerLane = kChunkElems / 4 / kBlock, kFlight = 8;
                static_assert(kPerLane % kFlight == 0, "chunk size and block size");
#pragma unroll
                for (int base = 0; base < kPerLane; base += kFlight) {
                    f32x4 g[kFlight], mp[kFlight];
#pragma unroll
                    for (int v = 0; v < kFlight; ++v) {
                        g[v] = load_grad4<BF16, true>(g0, (base + v) * kBlock + tid);
                        mp[v] = ld<true>(m4 + (base + v) * kBlock + tid);
                    }
#pragma unroll
                    for (int v = 0; v < kFlight; ++v) update4((base + v) * kBlock + tid, g[v], mp[v]);
                }
            } else {
                for (int j = tid; j < groups; j += kBlock) update4(j, load_grad4<BF16, true>(g0, j), ld<true>(m4 + j));
            }
            done = groups * 4;
        }
        for (int j = done + tid; j < len; j += kBlock) {
            float m_new;
            const double u = momentum_elem(h, mu, nesterov, load_grad1<BF16>(g0, j), m[j], &m_new);
            m[j] = m_new;
            acc = fma(u, u, acc);
        }
        const double s = wave_sum(acc);
        if ((tid & 63) == 0) wave_sums[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) {
            double b = wave_sums[0];
#pragma unroll
            for (int w = 1; w < kWavesPerBlock; ++w) b += wave_sums[w];
            t.partials[ck.slot] = b;
        }
        __syncthreads();
    }
}

// What a workgroup needs to know about matrix z of its batch.  The iteration runs on the wide orientation: X is mp x np, the
// transpose of a tall matrix.
struct MatrixView {
    uint32_t tensor;
    int64_t  rows, cols;
    double   scale;
    bool     tall;
};

__device__ __forceinline__ MatrixView matrix_view(const MuonMatrix* members, uint32_t z)
{
    const MuonMatrix* mm = members + z;
    const int64_t rows = uniform_load(&mm->rows), cols = uniform_load(&mm->cols);
    return {uniform_load(&mm->tensor), rows, cols, uniform_load(&mm->scale), rows > cols};
}

__device__ __forceinline__ bool is_aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// One 64 x 64 tile of X0.  The source U (rows x cols, recomputed from g and the updated momentum) is walked in tiles of
// its extent padded to multiples of 128; every element of the padded extent is written: zeros outside the matrix.
// x: the matrix's X, rows of ld_x elements: U as it is, or, of a tall matrix, its transpose, through LDS so that it is written
// along its rows.
// VEC (cols a multiple of 4, g and m aligned to their elements): a lane handles 4 consecutive elements of a
// row on the way in and 4 consecutive elements of a row of X on the way out: 16-byte loads, 8-byte stores.
template <bool BF16, bool VEC>
__device__ __forceinline__ void normalise_tile(uint16_t* tile, gcbytes g, gcfloat m, int64_t rows, int64_t cols, int64_t r0,
                                               int64_t c0, double h, double inv_denom, double mu, int nesterov, bool tall, uint16_t* x,
                                               int64_t ld_x)
{
    constexpr int kTileLd = VEC ? 68 : 66;                 // u16 per LDS row (VEC: rows stay 8-byte aligned)
    auto x0_bits = [&](float gv, float mv) {
        const double gh = h * (double)gv;
        const double u = nesterov ? gh + mu * (double)mv : (double)mv;         // m already holds this step's momentum
        return float_to_bf16_bits((float)(u * inv_denom));
    };
    if constexpr (VEC) {
        const int q = (threadIdx.x & 15) * 4, p = threadIdx.x >> 4;            // 16 lanes per row, 16 rows per pass
        f32x4 gv[4], mv[4];
        bool in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {                                          // all loads first
            const int64_t r = r0 + p + 16 * k, c = c0 + q;
            in[k] = r < rows && c < cols;
            if (!in[k]) continue;
            const int64_t j = r * cols + c;
            gv[k] = load_grad4<BF16, true>(g + j * (BF16 ? 2 : 4), 0);
            mv[k] = ld<true>((const ADAGC_GLOBAL f32x4_any*)(m + j));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int tr = p + 16 * k;
            u32x2 bits = {0u, 0u};
            if (in[k]) {
                bits.x = x0_bits(gv[k].x, mv[k].x) | (x0_bits(gv[k].y, mv[k].y) << 16);
                bits.y = x0_bits(gv[k].z, mv[k].z) | (x0_bits(gv[k].w, mv[k].w) << 16);
            }
            *reinterpret_cast<u32x2*>(tall ? &tile[tr * kTileLd + q] : x + (r0 + tr) * ld_x + c0 + q) = bits;
        }
        if (!tall) return;                                                     // the same for the whole workgroup
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int tc = p + 16 * k;                                         // column of the tile = row of X
            u32x2 bits;
            bits.x = (uint32_t)tile[(q + 0) * kTileLd + tc] | ((uint32_t)tile[(q + 1) * kTileLd + tc] << 16);
            bits.y = (uint32_t)tile[(q + 2) * kTileLd + tc] | ((uint32_t)tile[(q + 3) * kTileLd + tc] << 16);
            *reinterpret_cast<u32x2*>(x + (c0 + tc) * ld_x + r0 + q) = bits;
        }
    } else {
        const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
            const int64_t r = r0 + ty + 4 * k, c = c0 + tx;
            uint16_t bits = 0;
            if (r < rows && c < cols) {
                const int64_t j = r * cols + c;
                bits = (uint16_t)x0_bits(load_grad1<BF16>(g + j * (BF16 ? 2 : 4), 0), m[j]);
            }
            if (tall) tile[(ty + 4 * k) * kTileLd + tx] = bits;
            else x[r * ld_x + c] = bits;
        }
        if (!tall) return;
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
            const int64_t c = c0 + ty + 4 * k, r = r0 + tx;
            x[c * ld_x + r] = tile[tx * kTileLd + ty + 4 * k];
        }
    }
}

// A workgroup's matrix, and which of the matrix's workgroups it is.
struct MuonPlace {
    MatrixView mv;
    uint32_t   b;
    uint16_t*  x;
    int        mp, np;
};
__device__ __forceinline__ MuonPlace place_of(const MuonSpans& spans)
{
    int g = 0;
    while (g + 1 < spans.n && blockIdx.x >= spans.s[g + 1].first) ++g;
    const MuonSpan& s = spans.s[g];
    const uint32_t z = (blockIdx.x - s.first) / s.per_matrix;
    return {matrix_view(s.members, z), blockIdx.x - s.first - z * s.per_matrix, s.x + (int64_t)z * s.mp * s.np, s.mp, s.np};
}

// Workgroup b of a matrix: tile b.
template <bool BF16>
__global__ __launch_bounds__(256) void muon_normalise_kernel(DeviceTables t, MuonSpans spans, double mu, int nesterov)
{
    __shared__ __attribute__((aligned(8))) uint16_t tile[64 * 68];
    const MuonPlace at = place_of(spans);
    const MatrixView& mv = at.mv;
    const int mp = at.mp, np = at.np;
    uint16_t* const x = at.x;
    const TensorArgs ta = load_tensor(t.targs, mv.tensor);
    const uint32_t tile_cols = (uint32_t)((mv.tall ? mp : np) / 64);
    const int64_t r0 = (int64_t)(at.b / tile_cols) * 64, c0 = (int64_t)(at.b % tile_cols) * 64;
    const double h = uniform_load(t.coef64 + mv.tensor);
    // (with a division for each element 136 us for 85 M parameters, so 119; the two quotients differ in the last bit of a double, and X0 is bf16)
    const double inv_denom = 1.0 / (sqrt(uniform_load(t.sumsq + mv.tensor)) + 1e-7);
    const gcbytes g = (gcbytes)ta.grad;
    const gcfloat m = (gcfloat)ta.exp_avg;
    // the workspace is padded to 128 elements a row, so only the caller's arrays decide
    if (mv.cols % 4 == 0 && is_aligned(ta.grad, BF16 ? 2 : 4) && is_aligned(ta.exp_avg, 4))
        normalise_tile<BF16, true>(tile, g, m, mv.rows, mv.cols, r0, c0, h, inv_denom, mu, nesterov, mv.tall, x, np);
    else
        normalise_tile<BF16, false>(tile, g, m, mv.rows, mv.cols, r0, c0, h, inv_denom, mu, nesterov, mv.tall, x, np);
}

// theta <- theta - lr (wd theta + scale O), O being X (bf16, rows of np elements) or, of a tall matrix, its transpose.
// Workgroup b of a matrix: elements b * 4096 ..., whatever the row length (with a workgroup per row, a row of
// 768 kept 192 of 256 lanes busy with one access each); of a tall matrix tile b of 64 x 64, O through LDS.
// Where cols is a multiple of 4 and theta (and the copy) are aligned to their elements: 4 elements per lane and access.
constexpr int kApplyElems = 4096;
template <bool COPY>
__global__ __launch_bounds__(256) void muon_apply_kernel(DeviceTables t, MuonSpans spans, double lr, double wd)
{
    __shared__ __attribute__((aligned(8))) uint16_t tile[64 * 68];
    const MuonPlace at = place_of(spans);
    const MatrixView& mv = at.mv;
    const int np = at.np;
    const uint16_t* const x = at.x;
    const TensorArgs ta = load_tensor(t.targs, mv.tensor);
    const double scale = mv.scale;
    const bool vec = mv.cols % 4 == 0 && is_aligned(ta.param, 4) && (!COPY || is_aligned(ta.param_copy, 2));
    auto one = [&](float th_f, uint32_t o_bits) {
        const double th = (double)th_f;
        const double ov = (double)__uint_as_float(o_bits << 16);
        return (float)(th - lr * (wd * th + scale * ov));
    };
    auto four = [&](gfloat theta, gu16 copy, f32x4 th, uint32_t o0, uint32_t o1, uint32_t o2, uint32_t o3) {
        const f32x4 out = {one(th.x, o0), one(th.y, o1), one(th.z, o2), one(th.w, o3)};
        st<true>((ADAGC_GLOBAL f32x4_any*)theta, out);
        if constexpr (COPY) {
            u32x2 cw;
            cw.x = float_to_bf16_bits(out.x) | (float_to_bf16_bits(out.y) << 16);
            cw.y = float_to_bf16_bits(out.z) | (float_to_bf16_bits(out.w) << 16);
            st<true>((ADAGC_GLOBAL u32x2_any*)copy, cw);
        }
    };
    const int tid = threadIdx.x;
    if (mv.tall) {
        const int64_t tile_cols = (mv.cols + 63) / 64;
        const int64_t r0 = at.b / tile_cols * 64, c0 = at.b % tile_cols * 64;
        if (r0 >= mv.rows) return;
        const int q = (tid & 15) * 4, p = tid >> 4;                            // 16 lanes per row, 16 rows per pass
        const gfloat theta = (gfloat)ta.param + r0 * mv.cols + c0;
        const gu16 copy = COPY ? (gu16)ta.param_copy + r0 * mv.cols + c0 : nullptr;
        const int rows = (int)(mv.rows - r0 < 64 ? mv.rows - r0 : 64), cols = (int)(mv.cols - c0 < 64 ? mv.cols - c0 : 64);
        u32x2 ow[4];
        f32x4 th[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)                                            // column c0 + ... of theta, 4 of its rows
            ow[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(x + (c0 + p + 16 * k) * np + r0 + q));
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (p + 16 * k < rows && q < cols) th[k] = ld<true>((const ADAGC_GLOBAL f32x4_any*)(theta + (int64_t)(p + 16 * k) * mv.cols + q));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<u32x2*>(&tile[(p + 16 * k) * 68 + q]) = ow[k];
        __syncthreads();
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int r = p + 16 * k;
                const int64_t e = (int64_t)r * mv.cols + q;
                if (r < rows && q < cols)
                    four(theta + e, COPY ? copy + e : nullptr, th[k], tile[q * 68 + r], tile[(q + 1) * 68 + r], tile[(q + 2) * 68 + r], tile[(q + 3) * 68 + r]);
            }
        } else {
            const int c = tid & 63;
            for (int r = tid >> 6; r < rows; r += 4) {
                if (c >= cols) continue;
                const int64_t e = (int64_t)r * mv.cols + c;
                const float out = one(theta[e], tile[c * 68 + r]);
                theta[e] = out;
                if constexpr (COPY) copy[e] = (uint16_t)float_to_bf16_bits(out);
            }
        }
        return;
    }
    const int64_t numel = mv.rows * mv.cols, first = (int64_t)at.b * kApplyElems;
    if (first >= numel) return;
    const int len = numel - first < kApplyElems ? (int)(numel - first) : kApplyElems;
    const gfloat theta = (gfloat)ta.param + first;
    const gu16 copy = COPY ? (gu16)ta.param_copy + first : nullptr;
    const uint32_t cols = (uint32_t)mv.cols;
    const int64_t row0 = first / mv.cols;                           // the same in all lanes
    const uint32_t col0 = (uint32_t)(first - row0 * mv.cols);
    const uint16_t* o = x + row0 * np;
    if (vec) {
        constexpr int kPer = kApplyElems / 4 / 256;
        f32x4 th[kPer];
        u32x2 ow[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t e = (uint32_t)(u * 256 + tid) * 4u;
            if ((int)e >= len) continue;                            // len is a multiple of 4 here, as cols is
            const uint32_t q = col0 + e, r = q / cols, c = q - r * cols;
            th[u] = ld<true>((const ADAGC_GLOBAL f32x4_any*)(theta + e));
            ow[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(o + (int64_t)r * np + c));
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t e = (uint32_t)(u * 256 + tid) * 4u;
            if ((int)e >= len) continue;
            four(theta + e, COPY ? copy + e : nullptr, th[u], ow[u].x & 0xFFFFu, ow[u].x >> 16, ow[u].y & 0xFFFFu, ow[u].y >> 16);
        }
    } else {
        for (int e = tid; e < len; e += 256) {
            const uint32_t q = col0 + (uint32_t)e, r = q / cols, c = q - r * cols;
            const float out = one(theta[e], o[(int64_t)r * np + c]);
            theta[e] = out;
            if constexpr (COPY) copy[e] = (uint16_t)float_to_bf16_bits(out);
        }
    }
}

}  // namespace

hipError_t launch_muon_momentum(const DeviceTables& t, double mu, int nesterov, int grad_bf16, int grid, hipStream_t stream)
{
    if (grad_bf16) muon_momentum_kernel<true><<<dim3(grid), dim3(kBlock), 0, stream>>>(t, mu, nesterov);
    else muon_momentum_kernel<false><<<dim3(grid), dim3(kBlock), 0, stream>>>(t, mu, nesterov);
    return hipGetLastError();
}

int64_t muon_normalise_blocks(int mp, int np) { return (int64_t)(mp / 64) * (np / 64); }

hipError_t launch_muon_normalise(const DeviceTables& t, const MuonSpans& spans, double mu, int nesterov, int grad_bf16, hipStream_t stream)
{
    if (grad_bf16) muon_normalise_kernel<true><<<dim3(spans.workgroups), dim3(256), 0, stream>>>(t, spans, mu, nesterov);
    else muon_normalise_kernel<false><<<dim3(spans.workgroups), dim3(256), 0, stream>>>(t, spans, mu, nesterov);
    return hipGetLastError();
}

int64_t muon_apply_blocks(int64_t rows, int64_t cols)
{
    if (rows > cols) return ((rows + 63) / 64) * ((cols + 63) / 64);
    return (rows * cols + kApplyElems - 1) / kApplyElems;
}

hipError_t launch_muon_apply(const DeviceTables& t, const MuonSpans& spans, double lr, double wd, int with_copy, hipStream_t stream)
{
    if (with_copy) muon_apply_kernel<true><<<dim3(spans.workgroups), dim3(256), 0, stream>>>(t, spans, lr, wd);
    else muon_apply_kernel<false><<<dim3(spans.workgroups), dim3(256), 0, stream>>>(t, spans, lr, wd);
    return hipGetLastError();
}

}  // namespace adagc
