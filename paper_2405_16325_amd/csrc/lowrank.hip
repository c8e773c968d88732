// Adapter preparation for slope_spmm_fwd (Eq. 11) with many tokens: T = X L.
//
// The paper concatenates L to the sparse weight so that one vendor SpMM call yields [Y1 | Y2] and
// a second fused GEMM adds Y2 R.  Here the sparse kernel is simply extended by r more k-steps on
// dense MFMA (operands T and R as stored), so only the skinny product T = X L is a kernel of its
// own: the dense tile kernel with a plain epilogue on a k-contiguous copy of L, split over d_in
// while its tiles are too few to fill the chip; it is bound by reading X once.  With up to
// XL_SMALL_MAX_TOKENS tokens the split over d_in in spmm_stream.hip computes T instead, from L as
// stored.
#include "skinny.h"

namespace {

// the skinny products of layers whose extents are not multiples of 64
template <bool BKMAJOR, bool AKMAJOR>
__global__ void __launch_bounds__(SK_WAVES * 64) skinny_ragged_kernel(const bf16_t* __restrict__ B, int64_t ldb,
                                                                      const bf16_t* __restrict__ A, int64_t lda, int n,
                                                                      int m, int K, bf16_t* __restrict__ C) {
    __shared__ __align__(16) uint8_t smem[SK_LDS];
    const int tiles_m = (m + SK_BJ - 1) / SK_BJ;
    skinny_tile<BKMAJOR, AKMAJOR>(B, ldb, A, lda, n, m, 0, K, (int)(blockIdx.x / tiles_m) * SK_BI,
                                  (int)(blockIdx.x % tiles_m) * SK_BJ, C, nullptr, smem);
}

}  // namespace

hipError_t launch_skinny_ragged(const bf16_t* B, int64_t ldb, bool b_kmajor, const bf16_t* A, int64_t lda, bool a_kmajor,
                                int64_t n, int64_t m, int64_t K, bf16_t* C, hipStream_t s) {
    const int64_t tiles = ((m + SK_BJ - 1) / SK_BJ) * ((n + SK_BI - 1) / SK_BI);
    if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(SK_WAVES * 64);
    if (b_kmajor && a_kmajor)
        skinny_ragged_kernel<true, true><<<grid, block, 0, s>>>(B, ldb, A, lda, (int)n, (int)m, (int)K, C);
    else if (a_kmajor)
        skinny_ragged_kernel<false, true><<<grid, block, 0, s>>>(B, ldb, A, lda, (int)n, (int)m, (int)K, C);
    else
        skinny_ragged_kernel<false, false><<<grid, block, 0, s>>>(B, ldb, A, lda, (int)n, (int)m, (int)K, C);
    return hipGetLastError();
}

hipError_t launch_lowrank_prepare(const bf16_t* X, int64_t n, int64_t d_in, const bf16_t* L, int64_t r, bf16_t* T,
                                  bf16_t* Lt, float* partial_or_null, size_t partial_bytes, hipStream_t s) {
    // L[d_in, r] -> Lt[r, d_in] (16-byte accesses on both sides: 5120 x 64 7.8 -> 4.6 us against 2-byte ones)
    hipError_t e = launch_transpose(L, d_in, r, Lt, s);
    if (e != hipSuccess) return e;
    // T[n, r] = X[n, d_in] * Lt[r, d_in]^T
    return launch_dense_tn_plain(X, n, Lt, r, d_in, d_in, T, partial_or_null, partial_bytes, s);
}
