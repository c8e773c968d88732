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

inline int64_t skinny_tiles(int64_t n, int64_t m) { return ((m + SK_BJ - 1) / SK_BJ) * ((n + SK_BI - 1) / SK_BI); }
inline int64_t skinny_chunks(int64_t K) { return (K + 32 * SK_WAVES - 1) / (32 * SK_WAVES); }   // in a row per wavefront

template <bool PBK, bool PAK, bool QBK, bool QAK>
hipError_t launch_skinny_pair(const SkinnyProduct& p, const SkinnyProduct& q, hipStream_t s) {
    const int64_t tp = skinny_tiles(p.n, p.m), tq = skinny_tiles(q.n, q.m);
    if (tp + tq > 0x7FFFFFFF - GRID_ROW) return hipErrorInvalidValue;
    skinny_ragged_kernel<PBK, PAK, QBK, QAK><<<grid_of(tp + tq), dim3(SK_WAVES * 64), 0, s>>>(SkinnyGrid{p, (int)tp},
                                                                                                   SkinnyGrid{q, (int)tq});
    return hipGetLastError();
}

}  // namespace

// Whole k-steps have the choice: the tile kernels stream better, but want a k-contiguous copy of a k-major operand and, on
// few tiles, a second kernel for the sums over slabs; this one takes operands as stored in one launch, at about 1.3 us per
// chunk of 32 k that a wavefront walks and round of two workgroups per compute unit.
// A product by itself, `most` chunks in one round of per_round workgroups: 8 in 512 where it saves the copy and the second
// kernel (1024 x 2048, rank 64: X L 2.7 + 5.1 + 3.8 -> 10.7 us; in two rounds, 16384 x 1024, rank 96, the forward took 33.1 us,
// 27.0 with the tile kernel).  5 in 256 where there is no copy to save (dY R^T): with two workgroups per compute unit it
// takes 12 us where the tile kernel, then in one launch, takes 9 (3 chunks: 3890 x 768, rank 160; 16384 x 768, rank 64; but
// 1024 x 768, rank 64 6.5 against 7.7).
bool skinny_is_short(int64_t n, int64_t m, int64_t K, int most, int per_round) {
    return skinny_tiles(n, m) <= per_round && skinny_chunks(K) <= most;
}

// One of the four products of the gradient call, which replace ten launches by two (1024 tokens, 2048 x 2048, rank 64:
// 42 -> 21 us; 256 tokens, 2560 x 2560, rank 512, two rounds: the call 51.3 -> 40.3).
bool skinny_pair_is_short(int64_t n, int64_t m, int64_t K) { return skinny_chunks(K) * ((skinny_tiles(n, m) + 511) / 512) <= 10; }

hipError_t launch_skinny_factors(const SkinnyProduct& t, const SkinnyProduct& t2, hipStream_t s) {
    return launch_skinny_pair<false, true, false, false>(t, t2, s);
}

hipError_t launch_skinny_ragged(const SkinnyProduct& p, hipStream_t s) {
    return p.a_kmajor ? launch_skinny_factors(p, {}, s) : launch_skinny_factors({}, p, s);
}

hipError_t launch_skinny_gradients(const SkinnyProduct& dl, const SkinnyProduct& dr, hipStream_t s) {
    return launch_skinny_pair<true, true, true, true>(dl, dr, s);
}
