// Adapter preparation for slope_spmm_fwd (Eq. 11) with many tokens: T = X L.
//
// The paper concatenates L to the sparse weight so that one vendor SpMM call yields [Y1 | Y2] and
// a second fused GEMM adds Y2 R.  Here the sparse kernel is simply extended by r more k-steps on
// dense MFMA (operands T and R as stored), so only the skinny product T = X L is a kernel of its
// own: the dense tile kernel with a plain epilogue, L as stored, split over d_in while its tiles
// are too few to fill the chip; it is bound by reading X once.  With up to
// XL_SMALL_MAX_TOKENS tokens the split over d_in in spmm_stream.hip computes T instead, from L as
// stored.
#include "pipeline.h"
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

// Whole k-steps have the choice: the tile kernels stream better, but on few tiles of a long contraction need a second kernel for the
// sums over slabs; this one is one launch always, at about 1.3 us per chunk of 32 k that a wavefront walks and round of
// workgroups.
// A product by itself, on at most one round of workgroups.  Over 260 calls each of X L and of dY R^T the form taken is 0.1 % and 0.2 %
// slower than the better one in the mean.  us, the call, tile kernel / here:
//   X L, up to five chunks, six on 64 tiles and more: 1024 x 512, rank 64 11.35 / 10.8; 600 x 1088, rank 64 18.4 / 17.9; 4096 x 1280,
//     rank 64 (128 tiles) 19.6 / 17.6; 1024 x 1536, rank 64 (32 tiles) 17.3 / 18.3, rank 160 (96) 19.7 / 19.4; 1024 x 2048, rank 64
//     19.4 / 21.5; two rounds, 16384 x 512, rank 64 14.9 / 16.0;
//   dY R^T, one chunk, four of rank 32, whose A is half a tile: 1024 x 256, rank 64 9.1 / 8.9; 1024 x 512, rank 64 11.15 / 11.5; 1 x 768,
//     rank 32 10.5 / 9.6, 64 tokens 10.6 / 11.2, 520 12.6 / 12.4; 520 x 1536, rank 32 16.1 / 17.6.
bool skinny_is_short(int64_t n, int64_t m, int64_t K, bool a_kmajor) {
    const int64_t tiles = skinny_tiles(n, m);
    const int64_t most = a_kmajor ? (tiles < 64 ? 5 : 6) : (m <= 32 ? 4 : 1);
    return tiles <= RESIDENT && skinny_chunks(K) <= most;
}

// One of the four products of the gradient call, in pairs, which the tile kernels take in two launches or up to four.  In chunks x
// rounds of two workgroups per compute unit: up to six for the factors T and T2, five for the gradients dL and dR.  Over 420 calls of
// 1 to 2000 tokens, 256 to 2048 a side, the form taken is 1.3 % slower than the better one in the mean (with ten for all 3.7 %; fewer
// chunks pay at some ranks and token counts and not at others).  us, the call, tile kernels / here: 1280 x 1280, rank 32, 200 tokens
// 19.0 / 17.7; 1024 x 1024, rank 128, 4 tokens 14.6 / 13.4, 32 14.8 / 15.3; 512 x 512, rank 64, 1024 tokens 21.8 / 21.0; 2048 x 2048, rank
// 64, 1024 tokens 30.9 / 35.2; 256 x 256, rank 32, 1536 tokens 21.8 / 21.7, 2048 24.2 / 25.4.
bool skinny_pair_is_short(int64_t b, int64_t d_in, int64_t d_out, int64_t r) {
    auto cost = [](int64_t n, int64_t m, int64_t K) { return skinny_chunks(K) * ((skinny_tiles(n, m) + 2 * RESIDENT - 1) / (2 * RESIDENT)); };
    return cost(b, r, d_in) <= 6 && cost(b, r, d_out) <= 6 && cost(d_in, r, b) <= 5 && cost(r, d_out, b) <= 5;
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
