// Launchers of the Muon path (muon.hip, muon_gemm.hip), called from api.cpp.  Kept apart from adagc_internal.h, which
// holds what the streaming kernels of the AdaGC step are compiled from.
#ifndef ADAGC_MUON_INTERNAL_H
#define ADAGC_MUON_INTERNAL_H

#include <vector>

#include "adagc_internal.h"
#include "muon_plan.h"

namespace adagc {

// bf16 matrix-core GEMM of the Newton-Schulz iteration (muon_gemm.hip): C = bf16(alpha P Q^T + beta D), D given
// through its transpose Dt, result written row-major (C), transposed (Ct) or both; batch products of one shape per
// launch, matrix z of each array at base + z * stride elements.
hipError_t launch_gemm_nt_bf16(const void* P, int ldp, const void* Q, int ldq, int M, int N, int K, float alpha,
                               float beta, const void* Dt, int lddt, void* C, int ldc, void* Ct, int ldct,
                               hipStream_t stream, bool symmetric = false, int batch = 1, int64_t stride_p = 0,
                               int64_t stride_q = 0, int64_t stride_dt = 0, int64_t stride_c = 0, int64_t stride_ct = 0);

// A batch of matrices of one padded shape in the workspace, matrix z of every array at z times its size: X and the next X
// (mp x np), A and B (mp x mp), bf16.
struct MuonGroup {
    int       mp, np, count;
    uint16_t *x, *x2, *a, *b;
};
// A planned launch (muon_plan.h), its arrays in device memory.
struct MuonLaunch {
    int side, workgroups;
    std::vector<int> groups;
    const GemmItem*  items;
    const int32_t*   first;
};
hipError_t launch_muon_product(MuonProduct product, const MuonLaunch& l, const MuonGroup* groups, hipStream_t stream);

// One matrix of a batch, in device memory.
struct MuonMatrix {
    uint32_t tensor;      // its place in the list
    uint32_t pad;
    int64_t  rows, cols;
    double   scale;       // sqrt(max(1, rows / cols))
};

// The batches of a round, whose matrices share the launches of the kernels around the products: workgroups first ..., per_matrix for each
// matrix.  (48 matrices of GPT-2-small in three batches: X0 in three launches 93 + 41 + 17 us, in one 136; their update 119 + 45 + 17, 178.)
struct MuonSpan {
    const MuonMatrix* members;             // the batch's records, DEVICE
    uint16_t*         x;                   // matrix z at z * mp * np
    int               mp, np;
    uint32_t          first, per_matrix;
};
struct MuonSpans {
    MuonSpan s[kMaxGroups];
    int      n;
    uint32_t workgroups;
};
// Appends a batch of `count` matrices with so many workgroups each.
inline void add_span(MuonSpans& spans, const MuonMatrix* members, uint16_t* x, int mp, int np, int count, int64_t per_matrix)
{
    spans.s[spans.n++] = MuonSpan{members, x, mp, np, spans.workgroups, (uint32_t)per_matrix};
    spans.workgroups += (uint32_t)(per_matrix * count);
}

// Muon (muon.hip): momentum update with the clipped gradient and the partial sums of squares of U; X0 of a round's
// matrices into the padded workspace; their parameter update.
hipError_t launch_muon_momentum(const DeviceTables& t, double mu, int nesterov, int grad_bf16, int grid, hipStream_t stream);
int64_t muon_normalise_blocks(int mp, int np);
hipError_t launch_muon_normalise(const DeviceTables& t, const MuonSpans& spans, double mu, int nesterov, int grad_bf16, hipStream_t stream);
int64_t muon_apply_blocks(int64_t rows, int64_t cols);
hipError_t launch_muon_apply(const DeviceTables& t, const MuonSpans& spans, double lr, double wd, int with_copy, hipStream_t stream);

}  // namespace adagc
#endif
