// The planner's partitions of the transposed-weight product as plain C calls, for the launch-bounds models of
// tests/test_kernel_bounds.py (built with csrc/plan.cpp by g++, no device code).
#include "nmm_internal.h"

using namespace nmm;

extern "C" {

// out: rows per wave, row blocks, rows walked together, k per slice, slices, grid, tickets, workspace bytes
int plan_nt(int64_t M, int64_t K, int64_t N, int64_t out[8]) {
    NtPlan q;
    const nmm_status st = plan_gemv_nt(M, K, N, &q);
    const int64_t v[8] = {q.r, q.row_blocks, q.rgroup, q.slice_k, q.ks, q.grid, q.n_tickets, int64_t(q.ws_bytes)};
    for (int i = 0; i < 8; ++i) out[i] = v[i];
    return st;
}

// out: quads of x rows per block, blocks, 16-row tiles of Wt, groups in flight, rotation, row blocks, grid;
// 0 where the product is not the matrix cores'
int plan_nt_matrix_cores(int64_t M, int64_t K, int64_t N, int64_t ldx, int64_t ldw, int64_t out[7]) {
    GemvArgs a;
    a.M = M; a.K = K; a.N = N; a.dt = NMM_BF16; a.ldx = ldx; a.ldw = ldw; a.ldy = N;
    NtMfmaPlan q;
    if (!plan_mfma_nt(a, &q)) return 0;
    const int64_t v[7] = {q.xr, q.mblocks, q.nt, q.depth, q.rot, q.row_blocks, q.grid};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
    return 1;
}

int heads_take_matrix_cores(int64_t batch, int64_t M, int64_t K, int64_t N) { return heads_on_mfma(batch, M, K, N); }

}  // extern "C"
