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

// The skinny products of layers whose extents are not multiples of 64, and short ones, one or two of them in a launch (no
// tiles: none): each has a few dozen workgroups, so two run beside each other (1000 tokens, 1000 x 1000, rank 64:
// 5.5 + 6.3 and 6.8 + 6.9 us one after the other, 7.3 and 6.5 in pairs; the training step 67.8 -> 56.8).
struct SkinnyGrid { SkinnyProduct p; int tiles; };

template <bool BKMAJOR, bool AKMAJOR>
__device__ __forceinline__ void skinny_product_tile(const SkinnyProduct& p, int tile, uint8_t* smem) {
    const int tiles_m = ((int)p.m + SK_BJ - 1) / SK_BJ;
    skinny_tile<BKMAJOR, AKMAJOR>(p.B, p.ldb, p.A, p.lda, (int)p.n, (int)p.m, 0, (uint32_t)p.K, tile / tiles_m * SK_BI,
                                  tile % tiles_m * SK_BJ, p.C, nullptr, smem);
}

template <bool PBK, bool PAK, bool QBK, bool QAK>
__global__ void __launch_bounds__(SK_WAVES * 64) skinny_ragged_kernel(SkinnyGrid p, SkinnyGrid q) {
    __shared__ __align__(16) uint8_t smem[SK_LDS];
    const int b = (int)flat_block();
    if (b < p.tiles) skinny_product_tile<PBK, PAK>(p.p, b, smem);
    else if (b - p.tiles < q.tiles) skinny_product_tile<QBK, QAK>(q.p, b - p.tiles, smem);
}

inline int64_t skinny_tiles(const SkinnyProduct& p) { return ((p.m + SK_BJ - 1) / SK_BJ) * ((p.n + SK_BI - 1) / SK_BI); }

template <bool PBK, bool PAK, bool QBK, bool QAK>
hipError_t launch_skinny_pair(const SkinnyProduct& p, const SkinnyProduct& q, hipStream_t s) {
    const int64_t tp = skinny_tiles(p), tq = skinny_tiles(q);
    if (tp + tq > 0x7FFFFFFF - GRID_ROW) return hipErrorInvalidValue;
    skinny_ragged_kernel<PBK, PAK, QBK, QAK><<<grid_of(tp + tq), dim3(SK_WAVES * 64), 0, s>>>(SkinnyGrid{p, (int)tp},
                                                                                                   SkinnyGrid{q, (int)tq});
    return hipGetLastError();
}

}  // namespace

// Whole k-steps have the choice: the tile kernels stream better, but want a k-contiguous copy of a k-major operand and, on
// few tiles, a second kernel for the sums over slabs; this one takes operands as stored in one launch, at about 1.3 us per
// chunk of 32 k that a wavefront walks and round of two workgroups per compute unit.  `most` chunks: 8 where it saves the
// copy and the second kernel, 5 where the second kernel only, 10 for the pairs below (1024 tokens, 2048 x
// 2048, rank 64: X L 2.7 + 5.1 + 3.8 -> 10.7 us, the gradient call's adapter part 42 us in ten launches -> 21 in two).
bool skinny_is_short(int64_t n, int64_t m, int64_t K, int most) {
    const int64_t tiles = ((m + SK_BJ - 1) / SK_BJ) * ((n + SK_BI - 1) / SK_BI), steps = (K + 32 * SK_WAVES - 1) / (32 * SK_WAVES);
    return steps * ((tiles + 511) / 512) <= most;
}

hipError_t launch_skinny_factors(const SkinnyProduct& t, const SkinnyProduct& t2, hipStream_t s) {
    return launch_skinny_pair<false, true, false, false>(t, t2, s);
}

hipError_t launch_skinny_ragged(const SkinnyProduct& p, hipStream_t s) {
    return p.a_kmajor ? launch_skinny_factors(p, {}, s) : launch_skinny_factors({}, p, s);
}

hipError_t launch_skinny_gradients(const SkinnyProduct& dl, const SkinnyProduct& dr, hipStream_t s) {
    return launch_skinny_pair<true, true, true, true>(dl, dr, s);
}

hipError_t launch_lowrank_prepare(const bf16_t* X, int64_t n, int64_t d_in, const bf16_t* L, int64_t r, bf16_t* T,
                                  bf16_t* Lt, float* partial_or_null, size_t partial_bytes, hipStream_t s) {
    // L[d_in, r] -> Lt[r, d_in] (16-byte accesses on both sides: 5120 x 64 7.8 -> 4.6 us against 2-byte ones)
    hipError_t e = launch_transpose(L, d_in, r, Lt, s);
    if (e != hipSuccess) return e;
    // T[n, r] = X[n, d_in] * Lt[r, d_in]^T
    return launch_dense_tn_plain(X, n, Lt, r, d_in, d_in, T, partial_or_null, partial_bytes, s);
}
