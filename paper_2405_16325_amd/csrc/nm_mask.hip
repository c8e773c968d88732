// General N:M magnitude masks (Sec. 2.1; the paper's other patterns, e.g. 1:2 and 2:8 of Lemma 2.1)
// for M in {2, 4, 8} and any 1 <= N <= M.  Only 2:4 has a sparse MFMA, so these patterns run as
// masked dense weights ("emulation"): the kernels here emit the bit mask, the masked weight and,
// for the backward operand, its transpose; the products are plain dense tile kernels.
//
// Order inside a group: magnitude (bf16 bits with the sign cleared) descending, index ascending;
// positions outside the optional candidate mask never win and never count (double pruning:
// groups along the other axis, candidates = the first mask).
#include "common.h"

namespace {

// keep bits of one group: score[i] = candidate ? magnitude + 1 : 0
template <int M>
__device__ __forceinline__ uint32_t keep_of_group(const uint32_t (&score)[M], int n) {
    uint32_t keep = 0;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        uint32_t rank = 0;
#pragma unroll
        for (int j = 0; j < M; ++j)
            if (j != i) rank += (score[j] > score[i]) || (score[j] == score[i] && j < i);
        keep |= (uint32_t)(score[i] != 0u && rank < (uint32_t)n) << i;
    }
    return keep;
}

__device__ __forceinline__ uint32_t half_of(const u32x4& v, int e) { return (v[e >> 1] >> (16 * (e & 1))) & 0xFFFFu; }

// groups of M consecutive elements inside a row; one lane = 8 consecutive elements of a row, the lanes of
// a workgroup on consecutive chunks (mask and masked weight only: fully contiguous accesses); short-lived workgroups in
// address order, as in prune_rows_kernel
template <int M>
__global__ void __launch_bounds__(256) nm_mask_rows_kernel(const u32x4* __restrict__ W, size_t chunks, int n,
                                                           const uint8_t* __restrict__ cand,
                                                           uint8_t* __restrict__ mask, u32x4* __restrict__ masked) {
    const size_t c = (size_t)flat_block() * 256 + threadIdx.x;
    if (c >= chunks) return;
    const u32x4 v = W[c];
    const uint32_t cb = cand ? cand[c] : 0xFFu;
    uint32_t keep = 0;
#pragma unroll
    for (int g = 0; g < 8 / M; ++g) {
        uint32_t score[M];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            int e = g * M + i;
            score[i] = ((cb >> e) & 1u) ? (half_of(v, e) & 0x7FFFu) + 1u : 0u;
        }
        keep |= keep_of_group<M>(score, n) << (g * M);
    }
    mask[c] = (uint8_t)keep;
    u32x4 out;
#pragma unroll
    for (int w = 0; w < 4; ++w)
        out[w] = (((keep >> (2 * w)) & 1u) ? (v[w] & 0xFFFFu) : 0u) | (((keep >> (2 * w + 1)) & 1u) ? (v[w] & 0xFFFF0000u) : 0u);
    if (masked) masked[c] = out;
}

// The same with the transposed masked weight as a further output.
// A workgroup takes a tile of 64 columns x 128 rows (thread = chunk tx of 8 columns, rows ty + 32 i);
// the transposed masked weight, if asked for, leaves through LDS in runs of 128 rows per column.
template <int M>
__global__ void __launch_bounds__(256) nm_mask_rows_t_kernel(const bf16_t* __restrict__ W, int rows, int cols, int n,
                                                           const uint8_t* __restrict__ cand,
                                                           uint8_t* __restrict__ mask, bf16_t* __restrict__ masked,
                                                           bf16_t* __restrict__ masked_t) {
    constexpr int TR = 128, PITCH = TR + 2;
    __shared__ bf16_t tile[64 * PITCH];
    const size_t cpr = (size_t)cols / 8;
    const int tx = threadIdx.x & 7, ty = threadIdx.x >> 3;
    const size_t cc = (size_t)blockIdx.x * 8 + tx, r0 = (size_t)blockIdx.y * TR;
#pragma unroll
    for (int i = 0; i < TR / 32; ++i) {
        const size_t row = r0 + ty + 32 * i;
        if (cc >= cpr || row >= (size_t)rows) continue;
        const size_t c = row * cpr + cc;
        const u32x4 v = *(const u32x4*)(W + c * 8);
        const uint32_t cb = cand ? cand[c] : 0xFFu;
        uint32_t keep = 0;
#pragma unroll
        for (int g = 0; g < 8 / M; ++g) {
            uint32_t score[M];
#pragma unroll
            for (int q = 0; q < M; ++q) {
                int e = g * M + q;
                score[q] = ((cb >> e) & 1u) ? (half_of(v, e) & 0x7FFFu) + 1u : 0u;
            }
            keep |= keep_of_group<M>(score, n) << (g * M);
        }
        mask[c] = (uint8_t)keep;
        u32x4 out;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            out[w] = (((keep >> (2 * w)) & 1u) ? (v[w] & 0xFFFFu) : 0u) | (((keep >> (2 * w + 1)) & 1u) ? (v[w] & 0xFFFF0000u) : 0u);
        if (masked) *(u32x4*)(masked + c * 8) = out;
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[(tx * 8 + e) * PITCH + ty + 32 * i] = (bf16_t)half_of(out, e);
    }
    __syncthreads();
    const size_t c0 = (size_t)blockIdx.x * 64;
    for (int idx = threadIdx.x; idx < 64 * TR; idx += 256) {
        const int c = idx / TR, r = idx % TR;
        if (c0 + c >= (size_t)cols || r0 + r >= (size_t)rows) continue;
        masked_t[(c0 + c) * (size_t)rows + r0 + r] = tile[c * PITCH + r];
    }
}

// groups of M consecutive elements inside a column; one lane = 8 consecutive columns x the M rows of a group.
// A workgroup takes a tile of 64 columns x 64 rows (thread = chunk tx of 8 columns, row group ty), so that the
// transposed masked weight leaves through LDS in whole 128-byte lines (lane-sized pieces of 2 M bytes scattered over
// eight rows of the output made this kernel 3-8 x slower).  What bounds it on small weights is the ranking's chain of
// vector instructions: two neighbouring columns are ranked at once in the 16-bit halves of a register (key = magnitude
// + 1, 0 outside the candidates; one comparison per pair of rows serves both ranks), and 64 rows per tile give four
// times the workgroups of tiles of 32 groups (2:8 masks of 4096 x 1024: 14.8 -> 9.2 us).
template <int M>
__global__ void __launch_bounds__(512 / M) nm_mask_cols_kernel(const bf16_t* __restrict__ W, int rows, int cols, int n,
                                                           const uint8_t* __restrict__ cand,
                                                           uint8_t* __restrict__ mask, bf16_t* __restrict__ masked,
                                                           bf16_t* __restrict__ masked_t, unsigned tiles_x) {
    constexpr int TR = 64, THREADS = 512 / M;                 // rows of a tile
    __shared__ __align__(16) uint8_t tile[64 * TR * 2];       // [column][row]; the 16-byte pieces of column c rotated by c / 8
    const size_t cpr = (size_t)cols / 8;                      // 8-column chunks per row
    const int tx = threadIdx.x & 7, ty = threadIdx.x >> 3;
    const unsigned block = (unsigned)flat_block();
    const size_t tile_x = block % tiles_x, tile_y = block / tiles_x;
    if (tile_y * TR >= (size_t)rows) return;                  // past the last tile (uniform)
    const size_t cc = tile_x * 8 + tx;                        // chunk of 8 columns
    const size_t row0 = tile_y * TR + ty * M;                 // first row of the group
    const bool live = cc < cpr && row0 < (size_t)rows;        // rows % M == 0: a group is whole or absent
    u32x4 v[M];
    if (live) {
        uint32_t cb[M], keep[M];
#pragma unroll
        for (int k = 0; k < M; ++k) {
            v[k] = *(const u32x4*)(W + (row0 + k) * (size_t)cols + cc * 8);
            cb[k] = cand ? cand[(row0 + k) * cpr + cc] : 0xFFu;
            keep[k] = 0;
        }
        const uint32_t ones = 0x00010001u, quota = (uint32_t)n * ones;
#pragma unroll
        for (int q = 0; q < 4; ++q) {                         // columns 2 q (low halves) and 2 q + 1 (high halves)
            uint32_t key[M], rank[M];
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const uint32_t in = ((cb[k] >> (2 * q)) & 1u) | (((cb[k] >> (2 * q + 1)) & 1u) << 16);
                key[k] = ((v[k][q] & 0x7FFF7FFFu) + ones) & ((in << 16) - in);
                rank[k] = (uint32_t)k * ones;                 // as if everything in front were at least as large
            }
#pragma unroll
            for (int i = 0; i < M; ++i)
#pragma unroll
                for (int j = i + 1; j < M; ++j) {
                    const uint32_t c = pk_beats(key[j], key[i], ones);   // ties leave the lower index in front
                    rank[i] += c;
                    rank[j] -= c;
                }
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const uint32_t kept = pk_beats(quota, rank[k], ones) & pk_beats(key[k], 0u, ones);
                keep[k] |= ((kept & 1u) | ((kept >> 15) & 2u)) << (2 * q);
                v[k][q] &= (kept << 16) - kept;               // 1 -> 0xFFFF in either half
            }
        }
#pragma unroll
        for (int k = 0; k < M; ++k) {
            mask[(row0 + k) * cpr + cc] = (uint8_t)keep[k];
            if (masked) *(u32x4*)(masked + (row0 + k) * (size_t)cols + cc * 8) = v[k];
        }
    }
    if (!masked_t) return;                                    // uniform
    if (live) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {                         // the group's M values of column 8 tx + e, two rows per dword
            uint8_t* dst = tile + (tx * 8 + e) * (TR * 2) + ((ty * M * 2) ^ (tx * 16));
#pragma unroll
            for (int k = 0; k < M; k += 2)
                *(uint32_t*)(dst + 2 * k) =
                    __builtin_amdgcn_perm(v[k + 1][e >> 1], v[k][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
        }
    }
    __syncthreads();
    // column c of the tile = TR consecutive elements of row (c0 + c) of the transposed output
    const size_t c0 = tile_x * 64, r0 = tile_y * TR;
    if (rows % 8 == 0) {                                      // 16-byte aligned rows, pieces inside the row or outside as a whole
#pragma unroll
        for (int u = 0; u < 64 * 8 / THREADS; ++u) {
            const int idx = (int)threadIdx.x + u * THREADS, c = idx >> 3, p = idx & 7;
            if (c0 + c >= (size_t)cols || r0 + 8 * p >= (size_t)rows) continue;
            *(u32x4*)(masked_t + (c0 + c) * (size_t)rows + r0 + 8 * p) = *(const u32x4*)(tile + c * (TR * 2) + ((p ^ (c >> 3)) * 16));
        }
        return;
    }
    for (int idx = threadIdx.x; idx < 64 * (TR / 2); idx += THREADS) {
        const int c = idx / (TR / 2), p = idx % (TR / 2);
        if (c0 + c >= (size_t)cols || r0 + 2 * p >= (size_t)rows) continue;      // rows is even
        *(uint32_t*)(masked_t + (c0 + c) * (size_t)rows + r0 + 2 * p) =
            *(const uint32_t*)(tile + c * (TR * 2) + ((4 * p) ^ ((c >> 3) * 16)));
    }
}

template <int M>
hipError_t launch_m(const bf16_t* W, int64_t rows, int64_t cols, int n, int axis, const uint8_t* cand, uint8_t* mask,
                    bf16_t* masked, bf16_t* masked_t, hipStream_t s) {
    if (axis == 0 && masked_t)
        nm_mask_rows_t_kernel<M><<<dim3((unsigned)((cols + 63) / 64), (unsigned)((rows + 127) / 128)), dim3(256), 0, s>>>(
            W, (int)rows, (int)cols, n, cand, mask, masked, masked_t);
    else if (axis == 0) {
        const size_t chunks = (size_t)rows * (size_t)(cols / 8);
        const int64_t blocks = (int64_t)((chunks + 255) / 256);
        if (!grid_fits(blocks)) return hipErrorInvalidValue;
        nm_mask_rows_kernel<M><<<grid_of(blocks), dim3(256), 0, s>>>((const u32x4*)W, chunks, n, cand, mask,
                                                                          (u32x4*)masked);
    } else {
        const int64_t tiles_x = (cols + 63) / 64, tiles = tiles_x * ((rows + 63) / 64);
        if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
        nm_mask_cols_kernel<M><<<grid_of(tiles), dim3(512 / M), 0, s>>>(W, (int)rows, (int)cols, n, cand, mask, masked,
                                                                             masked_t, (unsigned)tiles_x);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_nm_mask(const bf16_t* W, int64_t rows, int64_t cols, int n, int m, int axis, const uint8_t* cand,
                          uint8_t* mask, bf16_t* masked, bf16_t* masked_t, hipStream_t s) {
    if (m == 2) return launch_m<2>(W, rows, cols, n, axis, cand, mask, masked, masked_t, s);
    if (m == 4) return launch_m<4>(W, rows, cols, n, axis, cand, mask, masked, masked_t, s);
    return launch_m<8>(W, rows, cols, n, axis, cand, mask, masked, masked_t, s);
}
