// Elementwise kernels of the Muon step with AdaGC's clipped gradient (Muon is the optimizer the paper pairs
// AdaGC with in "Optimizer Compatibility: Muon and Lion", Sec. 5.4; its rule is the published one, the paper
// prints none):
//
//   muon_momentum_kernel    per chunk:  M <- mu M + h g;  partial sum of squares of U
//                                       (U = h g + mu M in the Nesterov form, U = M otherwise)
//   muon_normalise_kernel   per batch:  X0 = bf16(U / (||U||_F + 1e-7)) of every matrix into the zero-padded workspace,
//                                       row-major and transposed (the matrix-core products want both, see muon_gemm.hip)
//   muon_apply_kernel       per batch:  theta <- theta - lr (wd theta + scale O) of every matrix, optional bf16 copy
//
// A batch is one launch of each, over all of its matrices: a matrix of a few hundred rows is read in two microseconds,
// less than a launch takes.  48 hidden matrices of GPT-2-small (85 M parameters, bf16 gradients, three batches): normalise
// 48 x 7.7 us -> 3 x 55 us (10 B per parameter, 5.2 TB/s), apply 48 x 6.0 us -> 3 x 59 us (12 B, 5.8 TB/s).  At Llama-3-8B
// shapes a matrix fills the chip by itself: 2.08 -> 1.94 ms and 1.54 -> 1.46 ms per 872 M parameters.
//
// The clip coefficient h of every tensor comes from the same norm and rule kernels as for AdamW and Lion
// (kernels.hip); the Newton-Schulz products run in muon_gemm.hip.  Arithmetic is double with one rounding per
// stored value, as in the other update kernels; reductions are in fixed order.

#include "muon_internal.h"

namespace adagc {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    uint32_t rounded = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? ((u >> 16) | 0x40u) : rounded;
}

template <bool BF16>
__device__ __forceinline__ float grad_at(const void* g, int64_t j)
{
    if constexpr (BF16) return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(g)[j] << 16);
    else return reinterpret_cast<const float*>(g)[j];
}

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
        const uint32_t c = t.schedule ? t.schedule[k] : k;     // the visiting order of the norm kernel (XCD-aware)
        const ChunkRef ck = t.chunks[c];
        const TensorArgs& ta = t.targs[ck.tensor];
        const int64_t first = (int64_t)ck.index * kChunkElems;
        const int64_t rest = ta.numel - first;
        const int len = rest < (int64_t)kChunkElems ? (int)rest : kChunkElems;
        const double h = t.coef64[ck.tensor];
        float* m = reinterpret_cast<float*>(ta.exp_avg) + first;
        double acc = 0.0;
        int done = 0;
        if (ta.vec_ok) {
            const int groups = len / 4;
            f32x4* m4 = reinterpret_cast<f32x4*>(m);
            auto load_g = [&](int j, float (&g)[4]) {
                if constexpr (BF16) {
                    const u32x2 w = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(ta.grad) + first) + j);
                    g[0] = __uint_as_float(w.x << 16);
                    g[1] = __uint_as_float(w.x & 0xFFFF0000u);
                    g[2] = __uint_as_float(w.y << 16);
                    g[3] = __uint_as_float(w.y & 0xFFFF0000u);
                } else {
                    const f32x4 w = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(ta.grad) + first) + j);
                    g[0] = w.x; g[1] = w.y; g[2] = w.z; g[3] = w.w;
                }
            };
            auto update4 = [&](int j, const float (&g)[4], const f32x4 mp) {
                f32x4 mn;
                float e;
                double u = momentum_elem(h, mu, nesterov, g[0], mp.x, &e); mn.x = e; acc = fma(u, u, acc);
                u = momentum_elem(h, mu, nesterov, g[1], mp.y, &e); mn.y = e; acc = fma(u, u, acc);
                u = momentum_elem(h, mu, nesterov, g[2], mp.z, &e); mn.z = e; acc = fma(u, u, acc);
                u = momentum_elem(h, mu, nesterov, g[3], mp.w, &e); mn.w = e; acc = fma(u, u, acc);
                __builtin_nontemporal_store(mn, m4 + j);
            };
            if (len == kChunkElems) {
                // a full chunk is 16 vectors per lane: 8 of each array in flight at a time
                constexpr int kPerLane = kChunkElems / 4 / kBlock, kFlight = 8;
                static_assert(kPerLane % kFlight == 0, "chunk size and block size");
#pragma unroll
                for (int base = 0; base < kPerLane; base += kFlight) {
                    float g[kFlight][4];
                    f32x4 mp[kFlight];
#pragma unroll
                    for (int v = 0; v < kFlight; ++v) {
                        load_g((base + v) * kBlock + tid, g[v]);
                        mp[v] = __builtin_nontemporal_load(m4 + (base + v) * kBlock + tid);
                    }
#pragma unroll
                    for (int v = 0; v < kFlight; ++v) update4((base + v) * kBlock + tid, g[v], mp[v]);
                }
            } else {
                for (int j = tid; j < groups; j += kBlock) {
                    float g[4];
                    load_g(j, g);
                    update4(j, g, __builtin_nontemporal_load(m4 + j));
                }
            }
            done = groups * 4;
        }
        for (int j = done + tid; j < len; j += kBlock) {
            float m_new;
            const double u = momentum_elem(h, mu, nesterov, grad_at<BF16>(ta.grad, first + j), m[j], &m_new);
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
            t.partials[c] = b;
        }
        __syncthreads();
    }
}

// What a workgroup needs to know about matrix z of its batch: the caller's arrays, and where the matrix lies in the
// workspace.  The iteration runs on the wide orientation: X is mp x np, Y = X^T; a tall matrix is its own Y.
struct MatrixView {
    uint32_t tensor;
    int64_t  rows, cols;
    bool     tall;
};

__device__ __forceinline__ MatrixView matrix_view(const MuonMatrix* members, uint32_t z)
{
    const MuonMatrix mm = members[z];
    return {mm.tensor, mm.rows, mm.cols, mm.rows > mm.cols};
}

__device__ __forceinline__ bool is_aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// One 64 x 64 tile of X0.  The source U (rows x cols, recomputed from g and the updated momentum) is walked in tiles of
// its extent padded to multiples of 128; every element of the padded extent is written: zeros outside the matrix.
// same[r][c] (leading dimension ld_same) receives the tile as is, trans[c][r] (ld_trans) its transpose, through LDS so
// that both are written along their rows.
// VEC (cols a multiple of 4, g and m 16-byte aligned; bf16 g 8-byte): a lane handles 4 consecutive elements of a
// row on the way in and 4 consecutive elements of a transposed row on the way out: 16-byte loads, 8-byte stores.
template <bool BF16, bool VEC>
__device__ __forceinline__ void normalise_tile(uint16_t* tile, const void* g, const float* m, int64_t rows, int64_t cols, int64_t r0,
                                               int64_t c0, double h, double denom, double mu, int nesterov, uint16_t* same,
                                               int64_t ld_same, uint16_t* trans, int64_t ld_trans)
{
    constexpr int kTileLd = VEC ? 68 : 66;                 // u16 per LDS row (VEC: rows stay 8-byte aligned)
    auto x0_bits = [&](float gv, float mv) {
        const double gh = h * (double)gv;
        const double u = nesterov ? gh + mu * (double)mv : (double)mv;         // m already holds this step's momentum
        return f32_to_bf16_bits((float)(u / denom));
    };
    if constexpr (VEC) {
        const int q = (threadIdx.x & 15) * 4, p = threadIdx.x >> 4;            // 16 lanes per row, 16 rows per pass
        float gv[4][4];
        f32x4 mv[4];
        bool in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {                                          // all loads first
            const int64_t r = r0 + p + 16 * k, c = c0 + q;
            in[k] = r < rows && c < cols;
            if (!in[k]) continue;
            const int64_t j = r * cols + c;
            if constexpr (BF16) {
                const u32x2 w = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(g) + j));
                gv[k][0] = __uint_as_float(w.x << 16);
                gv[k][1] = __uint_as_float(w.x & 0xFFFF0000u);
                gv[k][2] = __uint_as_float(w.y << 16);
                gv[k][3] = __uint_as_float(w.y & 0xFFFF0000u);
            } else {
                const f32x4 w = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g) + j));
                gv[k][0] = w.x; gv[k][1] = w.y; gv[k][2] = w.z; gv[k][3] = w.w;
            }
            mv[k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(m + j));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int tr = p + 16 * k;
            u32x2 bits = {0u, 0u};
            if (in[k]) {
                bits.x = x0_bits(gv[k][0], mv[k].x) | (x0_bits(gv[k][1], mv[k].y) << 16);
                bits.y = x0_bits(gv[k][2], mv[k].z) | (x0_bits(gv[k][3], mv[k].w) << 16);
            }
            *reinterpret_cast<u32x2*>(&tile[tr * kTileLd + q]) = bits;
            *reinterpret_cast<u32x2*>(same + (r0 + tr) * ld_same + c0 + q) = bits;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int tc = p + 16 * k;                                         // column of the tile = row of the transpose
            u32x2 bits;
            bits.x = (uint32_t)tile[(q + 0) * kTileLd + tc] | ((uint32_t)tile[(q + 1) * kTileLd + tc] << 16);
            bits.y = (uint32_t)tile[(q + 2) * kTileLd + tc] | ((uint32_t)tile[(q + 3) * kTileLd + tc] << 16);
            *reinterpret_cast<u32x2*>(trans + (c0 + tc) * ld_trans + r0 + q) = bits;
        }
    } else {
        const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
            const int64_t r = r0 + ty + 4 * k, c = c0 + tx;
            uint16_t bits = 0;
            if (r < rows && c < cols) {
                const int64_t j = r * cols + c;
                bits = (uint16_t)x0_bits(grad_at<BF16>(g, j), m[j]);
            }
            tile[(ty + 4 * k) * kTileLd + tx] = bits;
            same[r * ld_same + c] = bits;
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
            const int64_t c = c0 + ty + 4 * k, r = r0 + tx;
            trans[c * ld_trans + r] = tile[tx * kTileLd + ty + 4 * k];
        }
    }
}

// Workgroup (b, z): tile b of matrix z of the batch.  x, y: the batch's arrays, matrix z at z * mp * np.
template <bool BF16>
__global__ __launch_bounds__(256) void muon_normalise_kernel(DeviceTables t, const MuonMatrix* members, int mp, int np, double mu,
                                                              int nesterov, uint16_t* x, uint16_t* y)
{
    __shared__ __attribute__((aligned(8))) uint16_t tile[64 * 68];
    const MatrixView mv = matrix_view(members, blockIdx.y);
    const TensorArgs& ta = t.targs[mv.tensor];
    const uint32_t tile_cols = (uint32_t)((mv.tall ? mp : np) / 64);
    const int64_t r0 = (int64_t)(blockIdx.x / tile_cols) * 64, c0 = (int64_t)(blockIdx.x % tile_cols) * 64;
    const int64_t at = (int64_t)blockIdx.y * mp * np;
    uint16_t *same = (mv.tall ? y : x) + at, *trans = (mv.tall ? x : y) + at;
    const int64_t ld_same = mv.tall ? mp : np, ld_trans = mv.tall ? np : mp;
    const double h = t.coef64[mv.tensor];
    const double denom = sqrt(t.sumsq[mv.tensor]) + 1e-7;
    const float* m = static_cast<const float*>(ta.exp_avg);
    // the workspace is padded to 128 elements a row, so only the caller's arrays decide
    if (mv.cols % 4 == 0 && is_aligned(ta.grad, BF16 ? 8 : 16) && is_aligned(m, 16))
        normalise_tile<BF16, true>(tile, ta.grad, m, mv.rows, mv.cols, r0, c0, h, denom, mu, nesterov, same, ld_same, trans, ld_trans);
    else
        normalise_tile<BF16, false>(tile, ta.grad, m, mv.rows, mv.cols, r0, c0, h, denom, mu, nesterov, same, ld_same, trans, ld_trans);
}

// theta <- theta - lr (wd theta + scale O); workgroup (b, z): elements b * 4096 ... of matrix z of the batch, which O
// (bf16, rows of ld_o elements) holds row by row.
// 4096 elements per workgroup whatever the row length: with a workgroup per row, a row of 768 kept 192 of 256 lanes busy
// with one access each.
// VEC: cols is a multiple of 4 and theta (and the copy) are 16-byte (8-byte) aligned: 4 elements per lane and access.
constexpr int kApplyElems = 4096;
template <bool COPY>
__global__ __launch_bounds__(256) void muon_apply_kernel(DeviceTables t, const MuonMatrix* members, int mp, int np, const uint16_t* x,
                                                          const uint16_t* y, double lr, double wd)
{
    const MatrixView mv = matrix_view(members, blockIdx.y);
    const TensorArgs& ta = t.targs[mv.tensor];
    const int64_t numel = mv.rows * mv.cols, first = (int64_t)blockIdx.x * kApplyElems;
    if (first >= numel) return;
    const int len = numel - first < kApplyElems ? (int)(numel - first) : kApplyElems;
    const double scale = members[blockIdx.y].scale;
    const int64_t ld_o = mv.tall ? mp : np;
    const uint16_t* o = (mv.tall ? y : x) + (int64_t)blockIdx.y * mp * np;
    float* theta = static_cast<float*>(ta.param) + first;
    uint16_t* copy = COPY ? static_cast<uint16_t*>(ta.param_copy) + first : nullptr;
    const uint32_t cols = (uint32_t)mv.cols;
    const int64_t row0 = first / mv.cols;                           // the same in all lanes
    const uint32_t col0 = (uint32_t)(first - row0 * mv.cols);
    o += row0 * ld_o;
    auto one = [&](float th_f, uint32_t o_bits) {
        const double th = (double)th_f;
        const double ov = (double)__uint_as_float(o_bits << 16);
        return (float)(th - lr * (wd * th + scale * ov));
    };
    const int tid = threadIdx.x;
    if (cols % 4 == 0 && is_aligned(ta.param, 16) && (!COPY || is_aligned(ta.param_copy, 8))) {
        constexpr int kPer = kApplyElems / 4 / 256;
        f32x4 th[kPer];
        u32x2 ow[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t e = (uint32_t)(u * 256 + tid) * 4u;
            if ((int)e >= len) continue;                            // len is a multiple of 4 here, as cols is
            const uint32_t q = col0 + e, r = q / cols, c = q - r * cols;
            th[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(theta + e));
            ow[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(o + (int64_t)r * ld_o + c));
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t e = (uint32_t)(u * 256 + tid) * 4u;
            if ((int)e >= len) continue;
            f32x4 out;
            out.x = one(th[u].x, ow[u].x & 0xFFFFu);
            out.y = one(th[u].y, ow[u].x >> 16);
            out.z = one(th[u].z, ow[u].y & 0xFFFFu);
            out.w = one(th[u].w, ow[u].y >> 16);
            __builtin_nontemporal_store(out, reinterpret_cast<f32x4*>(theta + e));
            if constexpr (COPY) {
                u32x2 cw;
                cw.x = f32_to_bf16_bits(out.x) | (f32_to_bf16_bits(out.y) << 16);
                cw.y = f32_to_bf16_bits(out.z) | (f32_to_bf16_bits(out.w) << 16);
                __builtin_nontemporal_store(cw, reinterpret_cast<u32x2*>(copy + e));
            }
        }
    } else {
        for (int e = tid; e < len; e += 256) {
            const uint32_t q = col0 + (uint32_t)e, r = q / cols, c = q - r * cols;
            const float out = one(theta[e], o[(int64_t)r * ld_o + c]);
            theta[e] = out;
            if constexpr (COPY) copy[e] = (uint16_t)f32_to_bf16_bits(out);
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

hipError_t launch_muon_normalise(const DeviceTables& t, const MuonMatrix* members, int count, int mp, int np, double mu, int nesterov,
                                 int grad_bf16, uint16_t* x, uint16_t* y, hipStream_t stream)
{
    const dim3 grid((uint32_t)(mp / 64) * (uint32_t)(np / 64), (uint32_t)count);
    if (grad_bf16) muon_normalise_kernel<true><<<grid, dim3(256), 0, stream>>>(t, members, mp, np, mu, nesterov, x, y);
    else muon_normalise_kernel<false><<<grid, dim3(256), 0, stream>>>(t, members, mp, np, mu, nesterov, x, y);
    return hipGetLastError();
}

hipError_t launch_muon_apply(const DeviceTables& t, const MuonMatrix* members, int count, int64_t largest, int mp, int np,
                             const uint16_t* x, const uint16_t* y, double lr, double wd, int with_copy, hipStream_t stream)
{
    const dim3 grid((uint32_t)((largest + kApplyElems - 1) / kApplyElems), (uint32_t)count);
    if (with_copy) muon_apply_kernel<true><<<grid, dim3(256), 0, stream>>>(t, members, mp, np, x, y, lr, wd);
    else muon_apply_kernel<false><<<grid, dim3(256), 0, stream>>>(t, members, mp, np, x, y, lr, wd);
    return hipGetLastError();
}

}  // namespace adagc
